// nm_gemm for the calls the sparse-MFMA kernels do not take: widths K that are no multiple of 128,
// output counts that are no multiple of 4, buffers or leading dimensions without 16-byte alignment,
// and N >= 3 in the row layout.  Any pattern, any shape, any alignment, either layout.
//
// One workgroup of four wavefronts computes a BT-token x BO-row output tile, K in chunks of 256
// columns.  The packed weights are expanded once per tile to dense int8 rows in LDS and multiplied on
// the dense integer MFMA (v_mfma_i32_16x16x64_i8): at the widths that come here a call is bound by
// the latency of its few chunks (global -> registers -> LDS -> MFMA) and not by the matrix pipe, so
// the dense instruction's lower rate costs nothing, and one decode serves every pattern.  The next
// chunk's loads are in flight while the current one is multiplied; 35 KB of LDS (17 KB for the small
// tile) let several workgroups share a CU and cover each other's barriers.
//
// Loads are 16 bytes wide at any byte address (global memory takes unaligned vectors); only the chunk
// that holds a row's end is read in guarded pieces, so no byte past a row's K columns is touched.
// X is zero beyond K in LDS, which makes the columns of a partial chunk contribute nothing.
//
// Against one thread per output walking the metadata, which this kernel replaces: the 16 layers of a
// 312-wide encoder (F = 1200, 2:4 int8) at 1999 tokens 23.08 ms -> 0.139 ms a pass; eight layers of
// BERT-base at 3001 tokens with a 3-output layer behind them (K = 768, 31 tokens) 293.6 -> 112.0 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nm_internal.h"
#include "nm_gemm_common.h"

namespace nm {

namespace {

constexpr int KC = 256;                        // columns per chunk
constexpr int ROW = KC + 16;                   // LDS bytes per row: 16-byte reads of 8 consecutive rows cover all banks once

// The packed bytes of 32 consecutive columns of one weight row, and their expansion to 32 dense codes.
template <int N, int M, int BITS>
struct PackedUnit {
    using U = Unit<N, M, BITS>;
    static constexpr int VB = U::VBYTES, MB = U::MBYTES;
    uint32_t v[U::VD], m[U::MD];

    // UB bytes from `src`, of which `avail` are the row's own (the rest of the unit is zero)
    template <int UB, int WORDS>
    static __device__ __forceinline__ void read(const uint8_t* src, int avail, uint32_t (&dst)[WORDS])
    {
#pragma unroll
        for (int w = 0; w < WORDS; ++w) dst[w] = 0u;
        if (avail >= UB) {
            __builtin_memcpy(dst, src, UB);
            return;
        }
#pragma unroll
        for (int b = 0; b < UB; ++b)
            if (b < avail) dst[b / 4] |= (uint32_t)src[b] << (8 * (b % 4));
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
    __device__ __forceinline__ void load(const GemmArgs& a, int row, int unit)
    {
        if (a.pv.tiled) {
            const size_t block = (size_t)(row >> 4) * a.pv.slices + (unit >> 2);
            const int lane = (unit & 3) * 16 + (row & 15);
            read_pieces<VB>(a.vals + block * 64 * VB, lane, v);
            if constexpr (MB > 0) read_pieces<MB>(a.meta + block * 64 * MB, lane, m);
            return;
        }
        read<VB>(a.vals + (size_t)row * a.pv.stride + (size_t)unit * VB, (int)a.pv.stride - unit * VB, v);
        if constexpr (MB > 0) read<MB>(a.meta + (size_t)row * a.pm.stride + (size_t)unit * MB, (int)a.pm.stride - unit * MB, m);
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int w = 0; w < U::VD; ++w) v[w] = 0u;
#pragma unroll
        for (int w = 0; w < U::MD; ++w) m[w] = 0u;
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

// Columns k .. k+15 of a row of X, zero from column K on (K is a multiple of 4).
__device__ __forceinline__ v4i load_x16(const int8_t* row, int k, int K)
{
    v4i x = v4i{0, 0, 0, 0};
    if (k + 16 <= K) {
        __builtin_memcpy(&x, row + k, 16);
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (k + 4 * i < K) {
                int t;
                __builtin_memcpy(&t, row + k + 4 * i, 4);
                x[i] = t;
            }
    }
    return x;
}

template <int N, int M, int BITS, int BT, int BO>
__global__ void __launch_bounds__(256)
gemm_any_kernel(const GemmArgs a, const int tiles_o, const int n_tiles, const int vec)
{
    constexpr int FT = BT / 32, FO = BO / 32;          // 16x16 fragments per wavefront along each side (2 x 2 wavefronts)
    constexpr int XCH = BT * (KC / 16) / 256;          // 16-byte pieces of X per thread and chunk
    constexpr int WUN = BO * (KC / 32) / 256;          // weight units per thread and chunk
    static_assert(BT % 32 == 0 && BO % 32 == 0 && XCH * 256 == BT * (KC / 16) && WUN * 256 == BO * (KC / 32), "whole shares");
    __shared__ __align__(16) uint8_t xs[BT * ROW];
    __shared__ __align__(16) uint8_t ws[BO * ROW];

    // each XCD (workgroups are dealt to the eight in turn) takes a contiguous run of tiles
    const int per_xcd = (n_tiles + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= n_tiles) return;                       // whole workgroup leaves before any barrier
    const int t0 = (tile / tiles_o) * BT, o0 = (tile % tiles_o) * BO;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wt = wave & 1, wo = wave >> 1;
    const int li = lane & 15, lg = lane >> 4;

    v4i xr[XCH];
    PackedUnit<N, M, BITS> wr[WUN];
    auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < XCH; ++r) {
            const int c = tid + 256 * r;
            const int t = min(t0 + c / (KC / 16), a.tokens - 1);
            xr[r] = load_x16(a.X + (size_t)t * a.ldx, k0 + (c % (KC / 16)) * 16, a.K);
        }
#pragma unroll
        for (int r = 0; r < WUN; ++r) {
            const int u = tid + 256 * r;
            const int k = k0 + (u % (KC / 32)) * 32;
            if (k < a.K) wr[r].load(a, min(o0 + u / (KC / 32), a.O - 1), k / 32);
            else wr[r].clear();
        }
    };

    v4i acc[FO][FT];
#pragma unroll
    for (int fo = 0; fo < FO; ++fo)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) acc[fo][ft] = v4i{0, 0, 0, 0};

    load(0);
    for (int k0 = 0; k0 < a.K; k0 += KC) {
        if (k0 > 0) __syncthreads();                   // everyone has read the previous chunk
#pragma unroll
        for (int r = 0; r < XCH; ++r) {
            const int c = tid + 256 * r;
            *reinterpret_cast<v4i*>(xs + (c / (KC / 16)) * ROW + (c % (KC / 16)) * 16) = xr[r];
        }
#pragma unroll
        for (int r = 0; r < WUN; ++r) {
            const int u = tid + 256 * r;
            uint32_t d[8];
            wr[r].expand(d);
            v4i* dst = reinterpret_cast<v4i*>(ws + (u / (KC / 32)) * ROW + (u % (KC / 32)) * 32);
            dst[0] = v4i{(int)d[0], (int)d[1], (int)d[2], (int)d[3]};
            dst[1] = v4i{(int)d[4], (int)d[5], (int)d[6], (int)d[7]};
        }
        __syncthreads();
        if (k0 + KC < a.K) load(k0 + KC);
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

template <int N, int M, int BITS, int BT, int BO>
void launch_any_tile(const GemmArgs& a, long long tiles_t, long long tiles_o, bool vec, hipStream_t st)
{
    const long long n = tiles_t * tiles_o;
    hipLaunchKernelGGL((gemm_any_kernel<N, M, BITS, BT, BO>), dim3((unsigned)(8 * ((n + 7) / 8))), dim3(256), 0, st, a, (int)tiles_o, (int)n,
                       vec ? 1 : 0);
}

template <int N, int M, int BITS>
void launch_any(const GemmArgs& a_in, hipStream_t st)
{
    GemmArgs a = a_in;
    // a launch holds fewer than 2^32 threads: beyond 2^28 tokens (2^22 tiles of 64 along them) one per range
    constexpr int MOST = 1 << 28;
    if (a.tokens > MOST) {
        GemmArgs rest = a;
        const size_t esize = a.out_dtype == 1 ? 4 : a.out_dtype == 2 ? 2 : 1;
        rest.tokens -= MOST;
        rest.X += (size_t)MOST * a.ldx;
        if (a.acc) rest.acc += (size_t)MOST * a.ldo;
        if (a.out) rest.out = reinterpret_cast<uint8_t*>(a.out) + (size_t)MOST * a.ldo * esize;
        a.tokens = MOST;
        launch_any<N, M, BITS>(rest, st);
    }
    // Stores of four outputs at a time need rows of whole groups of four, all of them aligned.
    const bool vec = a.O % 4 == 0 && a.ldo % 4 == 0 && (uintptr_t)a.scales % 16 == 0 && (uintptr_t)a.bias % 16 == 0 &&
                     (uintptr_t)a.acc % 16 == 0 && (uintptr_t)a.out % 16 == 0;
    const long long big = ((a.tokens + 63ll) / 64) * ((a.O + 63ll) / 64);
    // Fewer than two 64 x 64 tiles per CU leave it short of wavefronts to cover the latency of a chunk.
    if (big < 512) launch_any_tile<N, M, BITS, 32, 32>(a, (a.tokens + 31ll) / 32, (a.O + 31ll) / 32, vec, st);
    else launch_any_tile<N, M, BITS, 64, 64>(a, (a.tokens + 63ll) / 64, (a.O + 63ll) / 64, vec, st);
}

}  // namespace

void launch_gemm_any(const GemmArgs& a, hipStream_t st)
{
#define NM_CASE(n, m) \
    if (a.N == n && a.M == m) return a.bits == 8 ? launch_any<n, m, 8>(a, st) : launch_any<n, m, 4>(a, st)
    NM_CASE(1, 4); NM_CASE(2, 4); NM_CASE(3, 4); NM_CASE(4, 4);
    NM_CASE(1, 8); NM_CASE(2, 8); NM_CASE(3, 8); NM_CASE(4, 8); NM_CASE(5, 8); NM_CASE(6, 8); NM_CASE(7, 8);
#undef NM_CASE
}

}  // namespace nm
