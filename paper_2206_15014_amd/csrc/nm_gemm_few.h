// nm_gemm on few tokens (tiled layout): problems of so few output tiles that the chip is idle and a
// launch is the latency of one walk along K.
//
// What bounds it: not bytes and not the matrix pipe (128 x 1024 -> 1024 reads 0.8 MB and multiplies for
// 0.1 us) but round trips.  A workgroup that walks K stage by stage through an LDS ring pays a barrier
// and a part of the memory latency per 128 columns, 32 times at K = 4096.  Here a workgroup of eight
// wavefronts owns a small tile and splits K: wavefront w takes the 128-column slices w, w + 8, ...,
// loads the fragments of up to four of them from global memory straight into registers (the tiled
// layout stores a weight fragment as the lanes read it), all in flight at once, and multiplies.  The
// eight partial tiles meet once, through LDS: int32 sums, so the order does not matter and the result
// is the same to the last bit.  One barrier per launch.
//
// Measured against the 64 x 48 tile with its LDS ring, which took these calls (2:4 int8, bf16 output,
// launches back to back, weights not in the L2s): 1 token 1024 -> 4096 4.78 -> 2.78 us, 4096 -> 1024
// 9.28 -> 3.23; 128 tokens 768 -> 768 4.29 -> 2.88, 1024 -> 4096 5.00 -> 4.24, 4096 -> 1024 9.43 -> 5.06;
// 512 tokens 1024 -> 1024 5.08 -> 3.93.  Dense int8, which had no small tile: 1 token 4096 -> 1024
// 15.40 -> 3.77, 128 tokens 768 -> 768 5.95 -> 3.00.
//
// Included behind the ring kernels of nm_gemm_dma.hip, not in front of them: see there.
#ifndef NM_GEMM_FEW_H
#define NM_GEMM_FEW_H

#include "nm_gemm_common.h"
#include "nm_gemm_sets.h"

namespace nm {
namespace {

constexpr int FEW_WAVES = 8;
// registers that the loads of a packed unit fill: a two-byte piece takes one like a dword
constexpr int load_registers(int bytes) { return bytes == 0 ? 0 : piece_bytes(bytes) == 2 ? bytes / 2 : (bytes + 3) / 4; }

template <int N, int M, int BITS, int FT, int FO>
__device__ __forceinline__ void gemm_few_tile(GemmArgs& a, const int tiles_t, const int tile)
{
    using U = Unit<N, M, BITS>;
    constexpr int NF = FT * FO;                // 16x16 fragments of the tile
    constexpr int VBLK = 64 * U::VBYTES, MBLK = 64 * U::MBYTES;
    static_assert(NF <= FEW_WAVES, "a wavefront finishes one fragment");
    __shared__ __align__(16) v4i part[FEW_WAVES * NF * 64];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int li = lane & 15, lg = lane >> 4;
    // outputs outermost: workgroups next to each other (on one XCD, see the callers) share weights
    const int t0 = (tile % tiles_t) * (16 * FT), o0 = (tile / tiles_t) * (16 * FO);
    const int nk = a.K >> 7, rb_last = (a.O + 15) / 16 - 1;

    const uint8_t* x[FT];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
        x[ft] = reinterpret_cast<const uint8_t*>(a.X) + (size_t)min(t0 + ft * 16 + li, a.tokens - 1) * a.ldx + lg * 16;
    const uint8_t* wv[FO];
    const uint8_t* wm[FO];
#pragma unroll
    for (int fo = 0; fo < FO; ++fo) {
        const size_t rb = (size_t)min(o0 / 16 + fo, rb_last) * nk;
        wv[fo] = a.vals + rb * VBLK;
        wm[fo] = a.meta + rb * MBLK;
    }

    v4i acc[FO][FT];
#pragma unroll
    for (int fo = 0; fo < FO; ++fo)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) acc[fo][ft] = v4i{0, 0, 0, 0};

    // slices first, first + 8, ... of this wavefront, CNT of them: loads of all, then products of all
    // slices a wavefront has in flight: two where their packed words would not fit the registers (5:8 int4 is the one of 10 + 10 bytes in
    // ten pieces: with four it spilled, 512 x 4096 -> 768 28.0 us, with two 14.0)
    constexpr int DEEP = FO * (load_registers(U::VBYTES) + load_registers(U::MBYTES)) > 24 ? 2 : 4;
    auto walk = [&](auto cnt, int first) __attribute__((always_inline)) {
        constexpr int CNT = decltype(cnt)::value;
        v8i b[CNT][FT];
        typename U::Raw w[CNT][FO];
#pragma unroll
        for (int i = 0; i < CNT; ++i) {
            const int k = min(first + i * FEW_WAVES, nk - 1);         // (a slice past the end is loaded and not used)
#pragma unroll
            for (int fo = 0; fo < FO; ++fo) w[i][fo] = U::load_tiled(wv[fo] + (size_t)k * VBLK, wm[fo] + (size_t)k * MBLK, lane);
#pragma unroll
            for (int ft = 0; ft < FT; ++ft) {
                const v4i lo = *reinterpret_cast<const v4i*>(x[ft] + (size_t)k * 128);
                const v4i hi = *reinterpret_cast<const v4i*>(x[ft] + (size_t)k * 128 + 64);
                b[i][ft] = v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
        }
        __builtin_amdgcn_sched_barrier(0);     // every load before the first product
#pragma unroll
        for (int i = 0; i < CNT; ++i) {
            if (first + i * FEW_WAVES >= nk) break;                   // uniform over the wavefront
#pragma unroll
            for (int fo = 0; fo < FO; ++fo) {
                if constexpr (U::DUAL) {
                    v4i c1, c2; int p1, p2;
                    U::template decode2<true>(w[i][fo], c1, p1, c2, p2);
#pragma unroll
                    for (int ft = 0; ft < FT; ++ft) {
                        acc[fo][ft] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(c1, b[i][ft], acc[fo][ft], p1, 0, 0);
                        acc[fo][ft] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(c2, b[i][ft], acc[fo][ft], p2, 0, 0);
                    }
                } else {
                    v4i codes; int pos;
                    U::template decode<true>(w[i][fo], codes, pos);
#pragma unroll
                    for (int ft = 0; ft < FT; ++ft)
                        acc[fo][ft] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(codes, b[i][ft], acc[fo][ft], pos, 0, 0);
                }
            }
        }
    };
    // scales and bias of the fragment this wavefront finishes: requested first, used last
    const int ff = wave < NF ? wave : 0, ffo = ff / FT, fft = ff % FT;
    float4 sw[1], bw[1];
    {
        const int o = min(o0 + ffo * 16 + 4 * lg, a.O - 4);
        sw[0] = *reinterpret_cast<const float4*>(a.scales + o);
        bw[0] = a.bias ? *reinterpret_cast<const float4*>(a.bias + o) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    a.act_scale = act_scale_of(a);
    a.act_scale_dev = nullptr;
    a.out_scale = out_scale_of(a);
    a.out_scale_dev = nullptr;

    if (nk <= FEW_WAVES) {
        walk(std::integral_constant<int, 1>{}, wave);
    } else if (DEEP == 2 || nk <= 2 * FEW_WAVES) {
        for (int k0 = 0; k0 < nk; k0 += 2 * FEW_WAVES) walk(std::integral_constant<int, 2>{}, k0 + wave);
    } else if (nk <= 3 * FEW_WAVES) {
        walk(std::integral_constant<int, (DEEP == 2 ? 2 : 3)>{}, wave);
    } else {
        for (int k0 = 0; k0 < nk; k0 += DEEP * FEW_WAVES) walk(std::integral_constant<int, DEEP>{}, k0 + wave);
    }

    unscale<BITS>(acc);
#pragma unroll
    for (int fo = 0; fo < FO; ++fo)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) part[(wave * NF + fo * FT + ft) * 64 + lane] = acc[fo][ft];
    __syncthreads();
    // The largest output: one commit per workgroup here too (layer chain 93 x 384, 2:4 int4, replayed 22.8 -> 17.3 us, 226 x 384, 1:8 int8 18.2 -> 16.9).
    // Not for two fragments: the two barriers cost what the one commit less saves (a maximum that is never reset: 140 calls 3 % slower).
    // Not for 5:8 int8 either: with it the compiler orders that pattern's loop so that 600 x 3072 -> 768 takes 12.8 us, without 11.3.
    // Any other output is done once it is stored, and its way out lies next to the stores: past the commit's instructions the last
    // fetch was one more trip to memory (0.25 us of 4.5 where other data has gone through the L2 since the last launch).
    const bool meet = NF > 2 && !(N == 5 && BITS == 8) && a.out_dtype == 3 && a.absmax != nullptr;
    if (wave >= NF && !meet) return;
    float m = 0.0f;
    if (wave < NF) {
        v4i sum[1][1] = {{v4i{0, 0, 0, 0}}};
#pragma unroll
        for (int w = 0; w < FEW_WAVES; ++w) sum[0][0] += part[(w * NF + ff) * 64 + lane];
        if (__builtin_expect(a.out_dtype == 3, 0)) {           // the columns' multipliers and offsets
            float g[4], h[4];
            requant_column(a.act_scale, sw[0].x, bw[0].x, a.out_scale, g[0], h[0]);
            requant_column(a.act_scale, sw[0].y, bw[0].y, a.out_scale, g[1], h[1]);
            requant_column(a.act_scale, sw[0].z, bw[0].z, a.out_scale, g[2], h[2]);
            requant_column(a.act_scale, sw[0].w, bw[0].w, a.out_scale, g[3], h[3]);
            sw[0] = make_float4(g[0], g[1], g[2], g[3]);
            bw[0] = make_float4(h[0], h[1], h[2], h[3]);
        }
        m = store_tile_pre<1, 1>(a, sum, sw, bw, o0 + ffo * 16, t0 + fft * 16, li, lg);
    }
    if (__builtin_expect(a.out_dtype != 3, 1)) return;
    if (meet) {
        __syncthreads();                       // every partial sum is read
        absmax_commit_group<FEW_WAVES>(m, out_scale_of(a), a.absmax, reinterpret_cast<float*>(part));
    } else {
        absmax_commit(m, out_scale_of(a), a.absmax);
    }
}

// One GEMM per launch; each XCD (workgroups are dealt to the eight in turn) takes a contiguous run of
// tiles, so that one XCD's L2 reads one share of the weights.
template <int N, int M, int BITS, int FT, int FO>
__global__ void __launch_bounds__(64 * FEW_WAVES)
gemm_few_kernel(const GemmArgs a_in, const int tiles_t, const int n_tiles)
{
    GemmArgs a = a_in;
    fetch_now(a);
    const int per_xcd = (n_tiles + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= n_tiles) return;               // whole workgroup leaves before the barrier
    gemm_few_tile<N, M, BITS, FT, FO>(a, tiles_t, tile);
}

// Several GEMMs per launch: here tiles_o[] holds the items' token tiles.
template <int N, int M, int BITS, int FT, int FO>
__global__ void __launch_bounds__(64 * FEW_WAVES)
gemm_few_batch_kernel(const GemmBatch p)
{
    const int n_tiles = p.first_tile[p.count];
    const int per_xcd = (n_tiles + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= n_tiles) return;
    int item = 0;                              // uniform over the workgroup
    while (item + 1 < p.count && tile >= p.first_tile[item + 1]) ++item;
    GemmArgs a = p.item[item];
    fetch_now(a);
    gemm_few_tile<N, M, BITS, FT, FO>(a, p.tiles_o[item], tile - p.first_tile[item]);
}

template <int N, int M, int BITS, int FT, int FO>
bool launch_few_tile(const GemmArgs* items, int count, hipStream_t st)
{
    GemmBatch b;
    b.count = count;
    b.first_tile[0] = 0;
    for (int i = 0; i < count; ++i) {
        const GemmArgs& a = items[i];
        const long long tt = (a.tokens + 16ll * FT - 1) / (16 * FT), n = tt * ((a.O + 16ll * FO - 1) / (16 * FO));
        if (b.first_tile[i] + n > (1 << 22)) return false;
        b.tiles_o[i] = (int)tt;
        b.first_tile[i + 1] = b.first_tile[i] + (int)n;
        b.item[i] = a;
    }
    for (int i = count; i < GEMM_BATCH_MAX; ++i) {      // unused slots: defined values
        b.item[i] = items[0];
        b.tiles_o[i] = 0;
        b.first_tile[i + 1] = b.first_tile[count];
    }
    if (planned_gemm()) return true;
    const int n_tiles = b.first_tile[count];
    const dim3 grid(8 * ((n_tiles + 7) / 8)), wg(64 * FEW_WAVES);
    if (count > 1) hipLaunchKernelGGL((gemm_few_batch_kernel<N, M, BITS, FT, FO>), grid, wg, 0, st, b);
    else hipLaunchKernelGGL((gemm_few_kernel<N, M, BITS, FT, FO>), grid, wg, 0, st, b.item[0], b.tiles_o[0], n_tiles);
    return true;
}

template <int N, int M, int BITS>
bool launch_few(const GemmArgs* items, int count, hipStream_t st, int cfg)
{
    note_gemm_tile(cfg);
    if (cfg == 141) return launch_few_tile<N, M, BITS, 1, 1>(items, count, st);
    if (cfg == 143) return launch_few_tile<N, M, BITS, 1, 2>(items, count, st);
    if (cfg == 142) return launch_few_tile<N, M, BITS, 2, 2>(items, count, st);
    if (cfg == 144) return launch_few_tile<N, M, BITS, 2, 4>(items, count, st);
    return false;
}

}  // namespace

// The patterns of this unit's set.  Returns true when it launched a kernel.
bool NM_SET_NAME(launch_gemm_few_set)(const GemmArgs* items, int count, hipStream_t st, int cfg)
{
    const GemmArgs& a = items[0];
#define NM_CASE(n, m, b) if (a.N == n && a.M == m && a.bits == b) return launch_few<n, m, b>(items, count, st, cfg)
    NM_SET_PATTERNS
#undef NM_CASE
    return false;
}

}  // namespace nm

#endif
