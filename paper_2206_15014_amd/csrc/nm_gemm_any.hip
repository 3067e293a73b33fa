// nm_gemm for the calls the sparse-MFMA kernels do not take: widths K that are no multiple of 128,
// output counts that are no multiple of 4, buffers or leading dimensions without 16-byte alignment,
// and N >= 3 in the row layout.  Any pattern, any shape, any alignment, either layout.
//
// One workgroup of four wavefronts computes a BT-token x BO-row output tile, K in chunks of 256
// columns.  A tile's packed weights go through registers to LDS: as operands of the sparse MFMA
// where a group keeps at most two (for 2:4 int8 the bytes as they are), expanded to dense int8 rows for
// the dense integer MFMA otherwise.  At the widths that come here a call is bound by the latency of
// its few chunks (global -> registers -> LDS -> MFMA) and not by the matrix pipe.  So two chunks are
// in flight, no load waits behind a branch that differs between lanes, and 15 KB of LDS (17 KB
// dense) for the small tile let several workgroups share a CU and cover each other's barriers.
//
// Loads are 16 bytes wide at any byte address (global memory takes unaligned vectors); only a buffer's
// last bytes are read in guarded pieces, so no byte past its end is touched.  X is zero beyond K in
// LDS, which makes the columns of a partial chunk contribute nothing, whatever the weights' bytes there.
//
// Outputs of very short rows, and of one to a few columns on many tokens, are computed by a thread each, walking the
// metadata (thread_per_output says when).  Against that, which took every call before: the 16 layers of a
// 312-wide encoder (F = 1200, 2:4 int8) at 1999 tokens 23.08 ms -> 0.106 ms a pass (0.139 with dense rows in LDS, one
// chunk in flight and the bytes of a row's last unit loaded one after the other); eight layers of BERT-base at 3001
// tokens with a 3-output layer behind them (K = 768, 31 tokens) 293.6 -> 112.0 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nm_internal.h"
#include "nm_gemm_common.h"

namespace nm {

namespace {

// A launch holds fewer than 2^32 threads: more tiles than this go in several, none of which can be too large, so a
// call is enqueued whole.  (Tiles are numbered in 32 bits: 2^31 of them would have outputs that no memory holds.)
constexpr long long ANY_LAUNCH_TILES = 1 << 23;
constexpr unsigned any_workgroups(long long tiles) { return (unsigned)(8 * ((tiles + 7) / 8)); }
static_assert((unsigned long long)any_workgroups(ANY_LAUNCH_TILES) * 256 < (1ull << 32), "threads of a launch");

constexpr int KC = 256;                        // columns per chunk

struct AnyPlan { int side; long long tiles_o, tiles; };        // of side x side outputs
AnyPlan any_plan(int tokens, int K, int O, int N, int M)
{
    const bool chunks = K > KC && (N < M || K >= 2 * KC);      // (dense: two whole ones; 1999 x 312 -> 872, 448 tiles: 6.6 us on the small tiles, 6.8)
    const long long big = ((tokens + 63ll) / 64) * ((O + 63ll) / 64);
    // Fewer than two 64 x 64 tiles per CU leave it short of wavefronts to cover the latency of a chunk.  With several chunks
    // the large tiles, which stage each operand half as often, are ahead from 400 on (2:4 int8, 1999 x 312 -> 936, 480 tiles: 7.0 -> 6.2 us,
    // 1700 x 1000 -> 1020, 432 tiles: 11.3 -> 9.5, 3:4 15.6 -> 13.2; 264 tiles, 1500 x 2720 -> 680, 1:4: 15.0 and 15.4; with one
    // chunk, dense, 2500 x 200 -> 696, 440 tiles: 5.7 and 5.1).
    const int side = big < (chunks ? 400 : 512) ? 32 : 64;
    const long long tiles_o = (O - 1ll + side) / side;
    return AnyPlan{side, tiles_o, ((tokens - 1ll + side) / side) * tiles_o};
}
AnyPlan any_plan(const GemmArgs& a) { return any_plan(a.tokens, a.K, a.O, a.N, a.M); }

constexpr int ROW = KC + 16;                   // LDS bytes per row: 16-byte reads of 8 consecutive rows cover all banks once
constexpr int CROW = KC / 2 + 16;              // the same for rows of sparse-MFMA codes (16 bytes per 32 columns) ...
constexpr int PROW = KC / 8 + 4;               // ... and of their positions (4 bytes per 32 columns)

// Where a chunk's loads go; the kernel and the check of its bounds on the host share these.  What a chunk loads past
// column K is dropped (X, in stage) or meets zeros of X (weights), so addresses are clamped to what the buffers hold and
// no load waits behind a branch of its lanes: pieces of X past K become the row's last columns, units past K the row's
// last unit.  Only a piece or unit that begins before a buffer's end and would reach past it is taken apart: the last
// token's, the last output row's.
__host__ __device__ inline int least(int a, int b) { return a < b ? a : b; }
__host__ __device__ inline bool x_whole(const GemmArgs& a, int t0, int side, int k0) { return k0 + KC <= a.K || (t0 < a.tokens - side && a.ldx >= 16); }      // (a piece may run into the next row)
__host__ __device__ inline bool w_whole(const GemmArgs& a, int o0, int side, int k0) { return k0 + KC <= a.K || (o0 < a.O - side && a.K >= 32); }
__host__ __device__ inline int x_row(const GemmArgs& a, int t0, int piece) { return least(t0 + piece / (KC / 16), a.tokens - 1); }
__host__ __device__ inline int x_column(const GemmArgs& a, int k) { return least(k, a.K - 4); }
__host__ __device__ inline int w_row(const GemmArgs& a, int o0, int unit) { return least(o0 + unit / (KC / 32), a.O - 1); }
__host__ __device__ inline int w_unit(const GemmArgs& a, int k0, int unit) { return least(k0 / 32 + unit % (KC / 32), (a.K - 1) / 32); }
__host__ __device__ inline size_t w_at_end(size_t at, size_t bytes, int unit_bytes) { return at + unit_bytes <= bytes ? at : bytes - unit_bytes; }

// The packed bytes of 32 consecutive columns of one weight row, and their expansion to 32 dense codes.
template <int N, int M, int BITS>
struct PackedUnit {
    using U = Unit<N, M, BITS>;
    static constexpr int VB = U::VBYTES, MB = U::MBYTES;
    uint32_t v[U::VD], m[U::MD];

    // UB bytes from byte `at` on of an array of `bytes` bytes, at least UB (the launcher sees to it); past its end, anything.
    template <int UB, int WORDS>
    static __device__ __forceinline__ void read_inside(const uint8_t* base, size_t at, uint32_t (&dst)[WORDS])
    {
        if constexpr (UB % 4 != 0) dst[WORDS - 1] = 0u;
        __builtin_memcpy(dst, base + at, UB);
    }
    template <int UB, int WORDS>
    static __device__ __forceinline__ void read_at_end(const uint8_t* base, size_t at, size_t bytes, uint32_t (&dst)[WORDS])
    {
#pragma unroll
        for (int w = 0; w < WORDS; ++w) dst[w] = 0u;
        // the array's last UB bytes at the most, moved down by as many as they begin too early
        const size_t from = w_at_end(at, bytes, UB);
        const int d = (int)(at - from);
        __builtin_memcpy(dst, base + from, UB);
#pragma unroll
        for (int step = 4; step >= 1; step /= 2)
#pragma unroll
            for (int w = 0; w < WORDS; ++w) dst[w] = (d / 4 & step) ? (w + step < WORDS ? dst[w + step] : 0u) : dst[w];
#pragma unroll
        for (int w = 0; w < WORDS; ++w) dst[w] = __builtin_amdgcn_alignbyte(w + 1 < WORDS ? dst[w + 1] : 0u, dst[w], (uint32_t)(d % 4));
    }
    template <int UB, int WORDS>
    static __device__ __forceinline__ void read_pieces(const uint8_t* block, int lane, uint32_t (&dst)[WORDS])
    {
        constexpr int PB = piece_bytes(UB);
#pragma unroll
        for (int w = 0; w < WORDS; ++w) dst[w] = 0u;
#pragma unroll
        for (int p = 0; p < UB / PB; ++p) __builtin_memcpy(reinterpret_cast<uint8_t*>(dst) + p * PB, block + (p * 64 + lane) * PB, PB);
    }
    __device__ __forceinline__ void load_tiled(const GemmArgs& a, int row, int unit)
    {
        const size_t block = (size_t)(row >> 4) * a.pv.slices + (unit >> 2);
        const int lane = (unit & 3) * 16 + (row & 15);
        read_pieces<VB>(a.vals + block * 64 * VB, lane, v);
        if constexpr (MB > 0) read_pieces<MB>(a.meta + block * 64 * MB, lane, m);
    }
    template <bool AT_END>
    __device__ __forceinline__ void load_rows(const GemmArgs& a, int row, int unit)
    {
        const size_t va = (size_t)row * a.pv.stride + (size_t)(unit * VB), ma = (size_t)row * a.pm.stride + (size_t)(unit * MB);
        if constexpr (AT_END) {
            read_at_end<VB>(a.vals, va, (size_t)a.O * a.pv.stride, v);
            if constexpr (MB > 0) read_at_end<MB>(a.meta, ma, (size_t)a.O * a.pm.stride, m);
        } else {
            read_inside<VB>(a.vals, va, v);
            if constexpr (MB > 0) read_inside<MB>(a.meta, ma, m);
        }
    }
    __device__ __forceinline__ void expand(uint32_t (&d)[8]) const
    {
        constexpr int EPU = U::EPU;
        uint32_t w[BITS == 8 ? U::VD : 2 * ((EPU + 7) / 8)];               // the codes as bytes, in entry order
        if constexpr (BITS == 8) {
#pragma unroll
            for (int i = 0; i < U::VD; ++i) w[i] = v[i];
        } else {
#pragma unroll
            for (int i = 0; i < (EPU + 7) / 8; ++i) {
                const uint32_t lo = sext4x4(v[i] & 0x0F0F0F0Fu), hi = sext4x4((v[i] >> 4) & 0x0F0F0F0Fu);
                w[2 * i] = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
                w[2 * i + 1] = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
            }
        }
        auto code = [&](int e) __attribute__((always_inline)) { return (w[e / 4] >> (8 * (e % 4))) & 0xFFu; };
        if constexpr (N == M) {
#pragma unroll
            for (int i = 0; i < 8; ++i) d[i] = w[i];
        } else if constexpr (M == 4) {
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                d[g] = 0u;
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const int e = g * N + j;
                    d[g] |= code(e) << (((m[e / 16] >> (2 * (e % 16))) & 3u) * 8u);
                }
            }
        } else {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint64_t x = 0;
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const int e = g * N + j;
                    x |= (uint64_t)code(e) << (((m[e / 8] >> (4 * (e % 8))) & 7u) * 8u);
                }
                d[2 * g] = (uint32_t)x;
                d[2 * g + 1] = (uint32_t)(x >> 32);
            }
        }
    }
};

template <int N, int M, int BITS, int BT, int BO>
__global__ void __launch_bounds__(256)
gemm_any_kernel(const GemmArgs a, const int tiles_o, const int first_tile, const int n_tiles, const int vec)
{
    constexpr int FT = BT / 32, FO = BO / 32;          // 16x16 fragments per wavefront along each side (2 x 2 wavefronts)
    constexpr int XCH = BT * (KC / 16) / 256;          // 16-byte pieces of X per thread and chunk
    constexpr int WUN = BO * (KC / 32) / 256;          // weight units per thread and chunk
    using U = Unit<N, M, BITS>;
    constexpr bool SPARSE = !U::DUAL;
    static_assert(BT % 32 == 0 && BO % 32 == 0 && XCH * 256 == BT * (KC / 16) && WUN * 256 == BO * (KC / 32), "whole shares");
    __shared__ __align__(16) uint8_t xs[BT * ROW];
    __shared__ __align__(16) uint8_t ws[BO * (SPARSE ? CROW + PROW : ROW)];

    // each XCD (workgroups are dealt to the eight in turn) takes a contiguous run of tiles
    const int per_xcd = (n_tiles + 7) >> 3;
    const int place = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (place >= n_tiles) return;                      // whole workgroup leaves before any barrier
    const int tile = first_tile + place;
    const int t0 = (tile / tiles_o) * BT, o0 = (tile % tiles_o) * BO;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wt = wave & 1, wo = wave >> 1;
    const int li = lane & 15, lg = lane >> 4;

    struct Chunk {
        v4i x[XCH];
        PackedUnit<N, M, BITS> w[WUN];
    };
    auto load = [&](int k0, Chunk& r) __attribute__((always_inline)) {
        if (k0 >= a.K) return;                         // this and all conditions below: uniform
        const bool xw = x_whole(a, t0, BT, k0), ww = w_whole(a, o0, BO, k0);
#pragma unroll
        for (int i = 0; i < XCH; ++i) {
            const int c = tid + 256 * i;
            const int8_t* row = a.X + (size_t)x_row(a, t0, c) * a.ldx;
            const int k = k0 + (c % (KC / 16)) * 16;
            if (xw) {
                __builtin_memcpy(&r.x[i], row + x_column(a, k), 16);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    int w;
                    __builtin_memcpy(&w, row + x_column(a, k + 4 * j), 4);
                    r.x[i][j] = w;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < WUN; ++i) {
            const int u = tid + 256 * i;
            const int row = w_row(a, o0, u), unit = w_unit(a, k0, u);
            if (a.pv.tiled) r.w[i].load_tiled(a, row, unit);
            else if (ww) r.w[i].template load_rows<false>(a, row, unit);
            else r.w[i].template load_rows<true>(a, row, unit);
        }
    };
    auto stage = [&](const Chunk& r, int k0) __attribute__((always_inline)) {
        const bool whole = k0 + KC <= a.K;             // uniform
#pragma unroll
        for (int i = 0; i < XCH; ++i) {
            const int c = tid + 256 * i;
            v4i x = r.x[i];
            if (!whole) {
                const int k = k0 + (c % (KC / 16)) * 16;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = k + 4 * j < a.K ? x[j] : 0;
            }
            *reinterpret_cast<v4i*>(xs + (c / (KC / 16)) * ROW + (c % (KC / 16)) * 16) = x;
        }
#pragma unroll
        for (int i = 0; i < WUN; ++i) {
            const int u = tid + 256 * i, row = u / (KC / 32), unit = u % (KC / 32);
            if constexpr (SPARSE) {
                typename U::Raw raw;
#pragma unroll
                for (int w = 0; w < U::VD; ++w) raw.v[w] = r.w[i].v[w];
#pragma unroll
                for (int w = 0; w < U::MD; ++w) raw.m[w] = r.w[i].m[w];
                v4i codes; int pos;
                U::decode(raw, codes, pos);
                *reinterpret_cast<v4i*>(ws + row * CROW + unit * 16) = codes;
                *reinterpret_cast<int*>(ws + BO * CROW + row * PROW + unit * 4) = pos;
            } else {
                uint32_t d[8];
                r.w[i].expand(d);
                v4i* dst = reinterpret_cast<v4i*>(ws + row * ROW + unit * 32);
                dst[0] = v4i{(int)d[0], (int)d[1], (int)d[2], (int)d[3]};
                dst[1] = v4i{(int)d[4], (int)d[5], (int)d[6], (int)d[7]};
            }
        }
    };

    v4i acc[FO][FT];
#pragma unroll
    for (int fo = 0; fo < FO; ++fo)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) acc[fo][ft] = v4i{0, 0, 0, 0};

    auto multiply = [&](int k0) __attribute__((always_inline)) {
        if constexpr (SPARSE) {
            const int steps = min((a.K - k0 + 127) >> 7, KC / 128);
            for (int s = 0; s < steps; ++s) {
                v8i xf[FT];
#pragma unroll
                for (int ft = 0; ft < FT; ++ft) {
                    const uint8_t* src = xs + (wt * (BT / 2) + ft * 16 + li) * ROW + s * 128 + lg * 16;
                    const v4i lo = *reinterpret_cast<const v4i*>(src), hi = *reinterpret_cast<const v4i*>(src + 64);
                    xf[ft] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                }
#pragma unroll
                for (int fo = 0; fo < FO; ++fo) {
                    const int row = wo * (BO / 2) + fo * 16 + li, unit = 4 * s + lg;
                    const v4i codes = *reinterpret_cast<const v4i*>(ws + row * CROW + unit * 16);
                    const int pos = *reinterpret_cast<const int*>(ws + BO * CROW + row * PROW + unit * 4);
#pragma unroll
                    for (int ft = 0; ft < FT; ++ft)
                        acc[fo][ft] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(codes, xf[ft], acc[fo][ft], pos, 0, 0);
                }
            }
        } else {
            const int steps = min((a.K - k0 + 63) >> 6, KC / 64);
            for (int s = 0; s < steps; ++s) {
                v4i xf[FT], wf[FO];
#pragma unroll
                for (int ft = 0; ft < FT; ++ft)
                    xf[ft] = *reinterpret_cast<const v4i*>(xs + (wt * (BT / 2) + ft * 16 + li) * ROW + s * 64 + lg * 16);
#pragma unroll
                for (int fo = 0; fo < FO; ++fo)
                    wf[fo] = *reinterpret_cast<const v4i*>(ws + (wo * (BO / 2) + fo * 16 + li) * ROW + s * 64 + lg * 16);
#pragma unroll
                for (int fo = 0; fo < FO; ++fo)
#pragma unroll
                    for (int ft = 0; ft < FT; ++ft)
                        acc[fo][ft] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[fo], xf[ft], acc[fo][ft], 0, 0, 0);
            }
        }
    };

    // two chunks in flight: a call of two chunks waits for memory once
    Chunk even, odd;
    load(0, even);
    load(KC, odd);
    for (int k0 = 0; k0 < a.K; k0 += 2 * KC) {
        if (k0 > 0) __syncthreads();                   // everyone has read the previous chunk
        stage(even, k0);
        __syncthreads();
        load(k0 + 2 * KC, even);
        multiply(k0);
        if (k0 + KC >= a.K) break;                     // uniform
        __syncthreads();
        stage(odd, k0 + KC);
        __syncthreads();
        load(k0 + 3 * KC, odd);
        multiply(k0 + KC);
    }

    // Lane (li, lg) holds rows 4*lg .. 4*lg+3 of token li of every fragment.
    if (vec) {                                         // whole, aligned groups of four outputs
        store_tile<FO, FT>(a, acc, o0 + wo * (BO / 2), t0 + wt * (BT / 2), li, lg);
        return;
    }
    const float s_act = act_scale_of(a), s_out = out_scale_of(a);
    float m = 0.0f;                                    // largest |code before rounding| (requantised output)
#pragma unroll
    for (int fo = 0; fo < FO; ++fo) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = o0 + wo * (BO / 2) + fo * 16 + 4 * lg + r;
            if (o >= a.O) continue;
            const float sw = a.scales[o], b = a.bias ? a.bias[o] : 0.0f;
            float g[4] = {0.f, 0.f, 0.f, 0.f}, h[4] = {0.f, 0.f, 0.f, 0.f};
            if (a.out_dtype == 3) requant_column(s_act, sw, b, s_out, g[0], h[0]);
#pragma unroll
            for (int ft = 0; ft < FT; ++ft) {
                const int t = t0 + wt * (BT / 2) + ft * 16 + li;
                if (t >= a.tokens) continue;
                const size_t at = (size_t)t * a.ldo + o;
                const int sum = acc[fo][ft][r];
                if (a.acc) a.acc[at] = sum;
                if (a.out_dtype == 3) {
                    reinterpret_cast<uint8_t*>(a.out)[at] = (uint8_t)requant4(v4i{sum, 0, 0, 0}, g, h, m);
                } else if (a.out_dtype != 0) {
                    const float y = (float)sum * (s_act * sw) + b;
                    if (a.out_dtype == 1) reinterpret_cast<float*>(a.out)[at] = y;
                    else reinterpret_cast<uint16_t*>(a.out)[at] = (uint16_t)pack_bf16x2(y, 0.0f);
                }
            }
        }
    }
    if (a.out_dtype == 3) absmax_commit(m, s_out, a.absmax);
}

// The smallest reductions: one thread per output, walking the metadata.  See thread_per_output.
__global__ void __launch_bounds__(256)
gemm_thread_kernel(const GemmArgs a, const long long first)
{
    const long long id_raw = first + (long long)blockIdx.x * 256 + threadIdx.x;
    const long long total = (long long)a.tokens * a.O;
    const bool live = id_raw < total;          // threads past the end recompute the last output and store nothing
    const long long id = live ? id_raw : total - 1;
    const int t = (int)(id / a.O), o = (int)(id % a.O);
    const int ib = (a.N >= a.M) ? 0 : (a.M == 4) ? 2 : 4;
    const int kc = a.K / a.M * a.N;
    const int8_t* x = a.X + (size_t)t * a.ldx;
    int sum = 0;
    for (int e = 0; e < kc; ++e) {
        int q, off;
        if (a.bits == 8) q = (int8_t)a.vals[a.pv.at((uint32_t)o, (uint32_t)e)];
        else { int nib = (a.vals[a.pv.at((uint32_t)o, (uint32_t)e >> 1)] >> ((e & 1) * 4)) & 15; q = (nib ^ 8) - 8; }
        if (ib == 0) off = e % a.N;
        else if (ib == 2) off = (a.meta[a.pm.at((uint32_t)o, (uint32_t)e >> 2)] >> ((e & 3) * 2)) & 3;
        else off = (a.meta[a.pm.at((uint32_t)o, (uint32_t)e >> 1)] >> ((e & 1) * 4)) & 15;
        sum += (int)x[(e / a.N) * a.M + off] * q;
    }
    const size_t at = (size_t)t * a.ldo + o;
    const float s_act = act_scale_of(a);
    if (a.out_dtype == 3) {                    // requantised output: every lane takes part in the reduction of max |y|
        const float s_out = out_scale_of(a);
        float g[4] = {0.f, 0.f, 0.f, 0.f}, h[4] = {0.f, 0.f, 0.f, 0.f};
        requant_column(s_act, a.scales[o], a.bias ? a.bias[o] : 0.0f, s_out, g[0], h[0]);
        float m = 0.0f;
        const uint32_t q = requant4(v4i{sum, 0, 0, 0}, g, h, m);
        if (live) reinterpret_cast<uint8_t*>(a.out)[at] = (uint8_t)q;
        absmax_commit(m, s_out, a.absmax);
        return;
    }
    if (!live) return;
    if (a.acc) a.acc[at] = sum;
    if (a.out_dtype != 0) {
        float y = (float)sum * (s_act * a.scales[o]) + (a.bias ? a.bias[o] : 0.0f);
        if (a.out_dtype == 1) reinterpret_cast<float*>(a.out)[at] = y;
        else reinterpret_cast<uint16_t*>(a.out)[at] = (uint16_t)pack_bf16x2(y, 0.0f);
    }
}

// Stores of four outputs at a time need rows of whole groups of four, all of them aligned.
bool whole_groups_of_four(const GemmArgs& a)
{
    return a.O % 4 == 0 && a.ldo % 4 == 0 && (uintptr_t)a.scales % 16 == 0 && (uintptr_t)a.bias % 16 == 0 &&
           (uintptr_t)a.acc % 16 == 0 && (uintptr_t)a.out % 16 == 0;
}

// Whether a thread per output is done sooner than tiles, from a duration model of both (microseconds, fitted to 2462 calls
// of 1 to 1000000 tokens, 1 to 1200 outputs and 1 to 40 kept entries a row; captured, operands in the caches).  A thread
// walks its row's kept entries one after the other: 0.27 us each (dense, without offsets, 0.2), and 1.65 us per million of
// them over the chip.  A tile costs its latency whatever it holds, and one of few columns is mostly padding.  So threads
// win on the shortest rows (2:8 int8, K = 8, 128 x 3: 2.8 us against 3.7; 2:4 int8, K = 8, 300 x 700 4.7 against 3.5) and on
// many tokens of a few outputs (2:4 int8, K = 24, 1000000 x 1: 22 against 74; 7:8 int8, K = 16: 24 against 152).
bool thread_per_output(const GemmArgs& a, bool vec)
{
    if ((long long)a.K * a.O < 32) return true;                                    // packed arrays shorter than a unit, which tiles do not read
    const double kept = (double)(a.K / a.M) * a.N, outputs = (double)a.tokens * a.O;
    if (kept > 128) return false;
    double thread = 2.15 + (a.N == a.M ? 0.2 : 0.27) * kept + 1.65e-6 * outputs * kept;
    double tile, more;                                                             // one round; each further 64 x 64 tile
    if (vec || a.O <= 16) {
        tile = a.O <= 2 ? 3.25 : !vec ? 3.5 : a.tokens < 16 ? 3.0 : 3.2;
        more = vec || a.O <= 4 ? 0.0048 : 0.0063;
    } else {                                                                       // single values stored side by side
        if (a.O > 64 && outputs > 1e6) return false;
        tile = (a.tokens < 16 ? 3.4 : a.tokens < 128 ? 3.75 : 4.1) + 4.2e-6 * outputs;
        more = 0.0015;
        thread += 2.6e-6 * outputs;
    }
    if (a.N >= 3 && a.N < a.M) {                                                   // the costlier expansions
        const bool costly = a.M == 4 || a.N != 4;
        tile += a.M == 4 ? (a.O <= 2 ? 0.55 : 0.2) : costly ? 0.7 : 0.1;
        more *= costly ? (a.M == 4 ? 1.45 : 2.0) : 1.15;
    }
    const double tiles = (double)((a.tokens - 1ll + 64) / 64) * (double)((a.O - 1ll + 64) / 64);
    return thread < tile + more * (tiles > 256.0 ? tiles - 256.0 : 0.0);
}

template <int N, int M, int BITS, int B>
void launch_any_tile(const GemmArgs& a, bool vec, hipStream_t st)
{
    const AnyPlan plan = any_plan(a);
    for (long long first = 0; first < plan.tiles; first += ANY_LAUNCH_TILES) {
        const int n = (int)(plan.tiles - first < ANY_LAUNCH_TILES ? plan.tiles - first : ANY_LAUNCH_TILES);
        hipLaunchKernelGGL((gemm_any_kernel<N, M, BITS, B, B>), dim3(any_workgroups(n)), dim3(256), 0, st, a, (int)plan.tiles_o, (int)first, n,
                           vec ? 1 : 0);
    }
}

template <int N, int M, int BITS>
void launch_any(const GemmArgs& a, hipStream_t st)
{
    const bool vec = whole_groups_of_four(a);
    if (any_plan(a).side == 32) launch_any_tile<N, M, BITS, 32>(a, vec, st);
    else launch_any_tile<N, M, BITS, 64>(a, vec, st);
}

}  // namespace

void launch_gemm_any(const GemmArgs& a, hipStream_t st)
{
    if (thread_per_output(a, whole_groups_of_four(a))) {
        const long long outputs = (long long)a.tokens * a.O, most = 1ll << 31;     // a launch holds fewer than 2^32 threads
        for (long long first = 0; first < outputs; first += most)
            hipLaunchKernelGGL(gemm_thread_kernel, dim3((unsigned)(((outputs - first < most ? outputs - first : most) + 255) / 256)), dim3(256), 0, st, a, first);
        return;
    }
#define NM_CASE(n, m) \
    if (a.N == n && a.M == m) return a.bits == 8 ? launch_any<n, m, 8>(a, st) : launch_any<n, m, 4>(a, st)
    NM_CASE(1, 4); NM_CASE(2, 4); NM_CASE(3, 4); NM_CASE(4, 4);
    NM_CASE(1, 8); NM_CASE(2, 8); NM_CASE(3, 8); NM_CASE(4, 8); NM_CASE(5, 8); NM_CASE(6, 8); NM_CASE(7, 8);
#undef NM_CASE
}

bool gemm_any_reads(const GemmArgs& a, size_t* x_end, size_t* v_end, size_t* m_end)
{
    if (thread_per_output(a, false)) return false;
    const AnyPlan plan = any_plan(a);
    const int side = plan.side;
    auto reach = [](size_t* end, size_t at, size_t bytes) { if (bytes && at + bytes > *end) *end = at + bytes; };
    auto unit_reach = [&](const PackedArray& p, size_t* end, int row, int unit, bool whole) {
        const size_t at = (size_t)row * p.stride + (size_t)unit * p.ub;
        if (p.ub == 0) return;
        if (p.tiled) reach(end, tiled_offset(row, unit * p.ub + p.ub - 1, p.ub, p.slices), 1);
        else reach(end, whole ? at : w_at_end(at, (size_t)a.O * p.stride, (int)p.ub), p.ub);
    };
    *x_end = *v_end = *m_end = 0;
    for (long long tile = 0; tile < plan.tiles; ++tile) {
        const int t0 = (int)(tile / plan.tiles_o) * side, o0 = (int)(tile % plan.tiles_o) * side;
        for (int k0 = 0; k0 < a.K; k0 += KC) {
            const bool xw = x_whole(a, t0, side, k0), ww = w_whole(a, o0, side, k0);
            for (int c = 0; c < side * (KC / 16); ++c)
                for (int j = 0; j < (xw ? 1 : 4); ++j)
                    reach(x_end, (size_t)x_row(a, t0, c) * a.ldx + x_column(a, k0 + (c % (KC / 16)) * 16 + 4 * j), xw ? 16 : 4);
            for (int u = 0; u < side * (KC / 32); ++u) {
                unit_reach(a.pv, v_end, w_row(a, o0, u), w_unit(a, k0, u), ww);
                unit_reach(a.pm, m_end, w_row(a, o0, u), w_unit(a, k0, u), ww);
            }
        }
    }
    return true;
}

int gemm_any_launches(int tokens, int K, int O, int N, int M, long long* tiles, unsigned* most_workgroups)
{
    const AnyPlan plan = any_plan(tokens, K, O, N, M);
    *tiles = plan.tiles;
    *most_workgroups = any_workgroups(plan.tiles < ANY_LAUNCH_TILES ? plan.tiles : ANY_LAUNCH_TILES);
    return (int)((plan.tiles + ANY_LAUNCH_TILES - 1) / ANY_LAUNCH_TILES);
}

}  // namespace nm
