// Projections of few rows with a long reduction (the text keys of a cross-attention: 154 x 1280 x 2048): bf16 MFMA GEMM with tiles of
// 32 rows, whose eight wavefronts each multiply the whole tile over K slices of their own.
//
// What bounds it: latency.  The chip has more CUs than larger tiles would give work to, and a tile's K loop is a string of
// steps that wait for operands: 64x128 tiles with the adapter's producers beside them are 30 workgroups of 33 steps.  Here
// 200 workgroups have four steps each, whose loads are in flight from the start on, and share nothing until the sums
// of their wavefronts meet in LDS.  No barriers in the K loop: a wavefront waits for its own loads only.
//
// LoRA: as in gemm16.hip the tile carries the rows of A as further columns, t = x A^T, and adds (scale t) B^T at the end;
// here every wavefront has a part of the sum over K of t too.
#include "gemm_dma.hpp"

namespace sd {

template <int V> using ThinInt = std::integral_constant<int, V>;

template <int BM, int BN, int RT>
struct TileThin {
    static constexpr int NW = 8;
    static constexpr int MI = BM / 16, NI = BN / 16, NB = MI * NI, NT = MI * RT;   // 16x16 blocks: of the tile, of t
    static constexpr int ROWS = BM + BN + 16 * RT;                   // of a slice: x, W, A
    static constexpr int LPT = ROWS / 8;                             // loads of a slice: 1 KB each, 8 rows of 128 bytes
    static constexpr int SLICE_CH = ROWS * 8;
    static constexpr int FIT = 160 * 64 / (NW * SLICE_CH);
    static constexpr int STAGES = FIT > 2 ? 2 : FIT;
    static constexpr int PER = (NB + NW - 1) / NW, TPER = (NT + NW - 1) / NW;      // blocks that a wavefront finishes
    // when the K loop is done: t in rows of nine chunks, and behind it the wavefronts' sums of t, then of the tile
    static constexpr int TP = 9, TTILE = RT ? BM * TP : 0, EXCH = NW * (NB > NT ? NB : NT) * 64;
    static constexpr int RING = NW * STAGES * SLICE_CH;
    static constexpr int LDS_CH = RING > TTILE + EXCH ? RING : TTILE + EXCH;
    static_assert(STAGES >= 1 && LDS_CH <= 160 * 64, "LDS");
};
constexpr int THIN_NONE = 0, THIN_BF16 = 1, THIN_F32 = 2;

template <int BM, int BN, int RT, int RES>
__global__ __launch_bounds__(512, 2) void gemm_thin_kernel(const GemmGroup g) {
    using T = TileThin<BM, BN, RT>;
    constexpr int NW = T::NW, MI = T::MI, NI = T::NI, LPT = T::LPT, SLICE = T::SLICE_CH, STAGES = T::STAGES;
    __shared__ u32x4 lds[T::LDS_CH];

    GemmProblem P;
    int tile, zero_n;
    int32_t* zero_ptr;
    if (!gemm_pick_tile(g, tile, P, zero_n, zero_ptr)) return;
    const int local = tile - P.tile_begin;
    const int band_tiles = 8 * P.tiles_n;
    const int band = local / band_tiles, rem = local - band * band_tiles;
    const int band_rows = min(8, P.tiles_m - band * 8);
    const int tn = rem / band_rows, tm = band * 8 + rem % band_rows;
    const int m0 = tm * BM, n0 = tn * BN;
    const int Mp = P.Mp, N = P.N, r = RT ? P.K1 : 0;
    const int nk = P.K0 / 64;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quad = lane >> 4;

    // ---- loader: a wavefront brings in all rows of its slices (rows past the end repeat the last one)
    uint32_t off[LPT];
    const char* const xbase = reinterpret_cast<const char*>(P.p0 + (int64_t)m0 * P.ldp0);
    const char* const wbase = reinterpret_cast<const char*>(P.q0 + (int64_t)n0 * P.ldq0);
    const char* const abase = reinterpret_cast<const char*>(r ? P.p1 : P.q0);   // (a projection without adapter in a launch that has some: rows of W, and nothing done with the product)
    const int xld = (int)P.ldp0 * 2, wld = (int)P.ldq0 * 2, ald = r ? (int)P.ldp1 * 2 : 0;
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int row = j * 8 + (lane >> 3);
        const int c16 = swz<8>(row, lane & 7) * 16;
        const bool isx = j < BM / 8, isa = j >= (BM + BN) / 8;
        const int k = min(row - (isx ? 0 : isa ? BM + BN : BM), isx ? Mp - 1 - m0 : isa ? (r ? r - 1 : 0) : N - 1 - n0);
        off[j] = (uint32_t)(k * (isx ? xld : isa ? ald : wld) + c16);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    const uint32_t mine = lds0 + wave * (STAGES * SLICE * 16);
    auto load = [&](int s, int stg) {
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const char* const b = j < BM / 8 ? xbase : j >= (BM + BN) / 8 ? abase : wbase;
            dma16_so<false>(b + (int64_t)s * 128, off[j], mine + (uint32_t)(stg * SLICE * 16 + j * 1024));
        }
    };
    // ---- prologue: the first slice, what the epilogue adds, the second slice
    if (wave < nk) load(wave, 0);
    // a wavefront finishes blocks wave, wave + 8, ...: row block b / NI and column block b % NI of the tile.  (Every lane loads, rows and
    // columns past the end their last ones)
    constexpr int PER = T::PER, KKT = RT > 2 ? 2 : 1;
    f32x4 resf[PER];
    u32x2 resb[PER], bias[PER];
    u32x4 bfrag[PER][KKT];                  // the block's rows of B, zeros past r
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int blk = min(wave + i * NW, T::NB - 1);
        const int mrow = m0 + blk / NI * 16 + l16, ncol = n0 + blk % NI * 16 + quad * 4;
        const int col = min(ncol, N - 4);
        const int64_t row = (int64_t)min(mrow, Mp - 1) * P.ldr;
        const uint32_t at = P.bias ? col : 0;
        bias[i] = *as_global(reinterpret_cast<const u32x2*>((P.bias ? P.bias : reinterpret_cast<const uint16_t*>(g_gemm_zeros)) + at));
        if (RES == THIN_F32) resf[i] = *as_global(reinterpret_cast<const f32x4*>(static_cast<const float*>(P.res) + row + col));
        if (RES == THIN_BF16) resb[i] = *as_global(reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(P.res) + row + col));
        if (RT)
#pragma unroll
            for (int kk = 0; kk < KKT; ++kk) {
                const uint16_t* src = P.q1 + (int64_t)min(n0 + blk % NI * 16 + l16, N - 1) * P.ldq1 + kk * 32 + quad * 8;
                if (kk * 32 + quad * 8 >= r) src = reinterpret_cast<const uint16_t*>(g_gemm_zeros);
                bfrag[i][kk] = *as_global(reinterpret_cast<const u32x4*>(src));
            }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (STAGES > 1 && wave + NW < nk) load(wave + NW, 1);
    __builtin_amdgcn_sched_barrier(0);

    f32x4 acc[MI][NI], acct[MI][RT ? RT : 1];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ri = 0; ri < RT; ++ri) acct[mi][ri] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int lsw = (l16 >> 1) & 7;
    const u32x4* const ring = lds + wave * (STAGES * SLICE) + l16 * 8;
    // The loads of slice s have landed when no more are in flight than the other slice's, issued behind them (loads retire in order).  The epilogue's
    // lie between the first slice's and the second's and are counted nowhere: however many the compiler makes of them, and wherever it puts them, a
    // wait is for slice s at the least.  (Against behind both slices, and counted: 0.95 to 1.02 of the time over
    // 1250 calls, at the median 0.99; with all operands from HBM 0.95 to 1.03, 1.00, where the first product waits for an adapter's rows of B too.)
    int st = 0;
#pragma unroll 1
    for (int s = wave; s < nk; s += NW) {
        if (STAGES > 1 && s + NW < nk) wait_vmcnt<LPT>();
        else wait_vmcnt<0>();
        bf16x8 xf[2][MI], wf[2][NI], rf[2][RT ? RT : 1];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const u32x4* const sx = ring + st * SLICE + ((kk * 4 + quad) ^ lsw);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) xf[kk][mi] = __builtin_bit_cast(bf16x8, sx[mi * 128]);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) wf[kk][ni] = __builtin_bit_cast(bf16x8, sx[(BM + ni * 16) * 8]);
#pragma unroll
            for (int ri = 0; ri < RT; ++ri) rf[kk][ri] = __builtin_bit_cast(bf16x8, sx[(BM + BN + ri * 16) * 8]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (s + STAGES * NW < nk) load(s + STAGES * NW, st);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[kk][ni], xf[kk][mi], acc[mi][ni], 0, 0, 0);
#pragma unroll
                for (int ri = 0; ri < RT; ++ri) acct[mi][ri] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rf[kk][ri], xf[kk][mi], acct[mi][ri], 0, 0, 0);
            }
        if (STAGES > 1) st ^= 1;
    }

    // ---- the wavefronts' sums meet: of t first, which is rounded to bf16, then of the tile
    uint16_t* const tb = reinterpret_cast<uint16_t*>(lds);
    f32x4* const ex = reinterpret_cast<f32x4*>(lds + T::TTILE) + lane;
    __syncthreads();
    if (RT && r) {
#pragma unroll
        for (int b = 0; b < T::NT; ++b) ex[(b * NW + wave) * 64] = acct[b / (RT ? RT : 1)][b % (RT ? RT : 1)];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < T::TPER; ++i) {
            const int b = wave + i * NW;
            if (b < T::NT) {
                f32x4 t = ex[b * NW * 64];
#pragma unroll
                for (int w = 1; w < NW; ++w) t += ex[(b * NW + w) * 64];
                const int col = b % (RT ? RT : 1) * 16 + quad * 4;
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)(col + e < r ? t[e] * P.t_scale : 0.f);
                *reinterpret_cast<bf16x4*>(tb + (b / (RT ? RT : 1) * 16 + l16) * (T::TP * 8) + col) = o;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int b = 0; b < T::NB; ++b) ex[(b * NW + wave) * 64] = acc[b / NI][b % NI];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int blk = wave + i * NW;
        if (blk >= T::NB) break;
        f32x4 v = ex[blk * NW * 64];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += ex[(blk * NW + w) * 64];
        if (RT && r)
#pragma unroll
            for (int kk = 0; kk < KKT; ++kk) {
                u32x4 tf = *reinterpret_cast<const u32x4*>(tb + (blk / NI * 16 + l16) * (T::TP * 8) + kk * 32 + quad * 8);
                if (RT == 1 && quad >= 2) tf = u32x4{0u, 0u, 0u, 0u};   // (one block of t: nothing has written the k-step's upper half)
                v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bfrag[i][kk]), __builtin_bit_cast(bf16x8, tf), v, 0, 0, 0);
            }
        // bias, residual, store
        const int mrow = m0 + blk / NI * 16 + l16, ncol = n0 + blk % NI * 16 + quad * 4;
        v[0] = P.alpha * v[0] + bf16lo_to_f32(bias[i][0]);
        v[1] = P.alpha * v[1] + bf16hi_to_f32(bias[i][0]);
        v[2] = P.alpha * v[2] + bf16lo_to_f32(bias[i][1]);
        v[3] = P.alpha * v[3] + bf16hi_to_f32(bias[i][1]);
        if (RES == THIN_F32) v += resf[i];
        if (RES == THIN_BF16) {
            v[0] += bf16lo_to_f32(resb[i][0]); v[1] += bf16hi_to_f32(resb[i][0]);
            v[2] += bf16lo_to_f32(resb[i][1]); v[3] += bf16hi_to_f32(resb[i][1]);
        }
        if (mrow >= Mp || ncol >= N) continue;
        if (RES != THIN_BF16 && P.y_f32) {
            *as_global(reinterpret_cast<f32x4*>(static_cast<float*>(P.y) + (int64_t)mrow * P.ldy + ncol)) = v;
            continue;
        }
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)v[e];
        if (RES == THIN_NONE && P.bias_on_rows == 2) {
#pragma unroll
            for (int e = 0; e < 4; ++e) *as_global(static_cast<__bf16*>(P.y) + (int64_t)(ncol + e) * P.ldy + mrow) = o[e];
        } else {
            *as_global(reinterpret_cast<bf16x4*>(static_cast<uint16_t*>(P.y) + (int64_t)mrow * P.ldy + ncol)) = o;
        }
    }
}

template <int BM, int BN, int RT>
static int launch_t(GemmGroup& g, hipStream_t stream) {
    using T = TileThin<BM, BN, RT>;
    int total = 0;
    g.n_lead = 0;
    g.zero_n = 0;
    for (int i = 0; i < g.n; ++i) {
        GemmProblem& P = g.p[i];
        P.tiles_m = (P.Mp + BM - 1) / BM;
        P.tiles_n = (P.N + BN - 1) / BN;
        P.tile_begin = total;
        g.first_tile[i] = total;
        total += P.tiles_m * P.tiles_n;
    }
    g.total_tiles = total;
    if (total == 0 || SD_DRY_RUN("thin %dx%d/%d%s; ", BM, BN, RT, dry_detail(", %d problems", g.n))) return SD_OK;
    const dim3 grid((total + 7) & ~7), block(64 * T::NW);
    if (!g.p[0].res) hipLaunchKernelGGL((gemm_thin_kernel<BM, BN, RT, THIN_NONE>), grid, block, 0, stream, g);
    else if (g.p[0].res_f32) hipLaunchKernelGGL((gemm_thin_kernel<BM, BN, RT, THIN_F32>), grid, block, 0, stream, g);
    else hipLaunchKernelGGL((gemm_thin_kernel<BM, BN, RT, THIN_BF16>), grid, block, 0, stream, g);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}
// size: 0 to 2, tiles of 32x32, 32x64 and 64x64, with ranks above 32 64x32 (what LDS holds of eight wavefronts' slices)
int launch_gemm_thin(GemmGroup& g, int size, hipStream_t stream) {
    int rmax = 0;
    for (int i = 0; i < g.n; ++i) rmax = g.p[i].K1 > rmax ? g.p[i].K1 : rmax;
    if (rmax > 32) return size == 0 ? launch_t<32, 32, 4>(g, stream) : launch_t<64, 32, 4>(g, stream);
    if (size == 0) return rmax == 0 ? launch_t<32, 32, 0>(g, stream) : rmax <= 16 ? launch_t<32, 32, 1>(g, stream) : launch_t<32, 32, 2>(g, stream);
    if (size == 1) return rmax == 0 ? launch_t<32, 64, 0>(g, stream) : rmax <= 16 ? launch_t<32, 64, 1>(g, stream) : launch_t<32, 64, 2>(g, stream);
    return rmax == 0 ? launch_t<64, 64, 0>(g, stream) : rmax <= 16 ? launch_t<64, 64, 1>(g, stream) : launch_t<64, 64, 2>(g, stream);
}

}  // namespace sd
