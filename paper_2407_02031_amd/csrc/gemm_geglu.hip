// The feed-forward in-projection, y = value * gelu(gate) of x W^T (+ adapter) with W [2F, K], in
// tiles of 160 output columns (320 rows of W) and 256 or 128 rows.
//
// What bounds it: the MFMAs of the most loaded CU.  The block's widths (2F = 5120 and 10240) are
// whole multiples of 320 columns, and its token counts make a whole number of rounds over 256 CUs
// of such tiles (8192x5120: two, 2048x10240: one) where 256x256 tiles need 2.5 and 1.25, that is
// three and two.  One workgroup per CU, eight wavefronts of 64x160 (or 32x160): 14 operand
// fragments per 40 MFMAs (12 per 20), 142 (or 91) FLOP per byte from L2.
//
// Two stages of 64 deep operand tiles fill the LDS, so a stage is refilled as soon as the last
// fragments of its tile are in registers, one load behind each of the next slots' MFMAs, and has the
// rest of the step to arrive.
//
// The chip lowers its clock under MFMAs (2.4 GHz idle, 1.75 in this main loop, whose matrix cores are then 83 % busy), so what
// an MFMA costs in energy is what it costs in time.  16x16x32 MFMAs take less of it than 32x32x16: the same
// 64x160 products on normal operands out of registers 2100 TFLOP/s against 1850, out of LDS 1860 against 1680.  In this kernel: 8192x5120x640 + 64 68.5 -> 64.5 us,
// 2048x10240x1280 + 64 54.0 -> 48.4, 988x10240x1280 30.1 -> 28.4 (with the weights from the last-level cache or HBM).
//
// The MFMA takes the rows of W first: a lane holds one row of x and four rows of W in a block of 16.  Blocks of value rows and of
// the gate rows of the same output columns take turns: GEGLU is done in the lane, and it stores four columns.
#include "gemm_dma.hpp"

namespace sd {

constexpr int GG_BN = 320, GG_OUT = 160, GG_WB = 10, GG_NW = 8;

// MI: 32 rows of x per wavefront times this; four wavefronts by rows, two by columns
template <int MI>
__global__ __launch_bounds__(512, 2) void gemm_geglu_kernel(const GemmGroup g) {
    constexpr int BM = MI * 128, XB = MI * 2, WB = GG_WB, NW = GG_NW;   // 16-row blocks of x and of W per wavefront
    constexpr int ROWS = BM + GG_BN, STAGE = ROWS * 8;         // 16-byte chunks of a stage
    constexpr int LPT = ROWS / 8 / NW, JP = BM / 8 / NW;       // loads per wavefront and stage, and those of x among them
    constexpr int SLOTS = 2 * WB;                              // a tile is two 32 deep k-steps of WB blocks of W; a slot multiplies one block by the x blocks
    constexpr int RING = MI == 2 ? 4 : 10;                     // blocks of W in registers (five where the accumulators are 160 registers: spills)
    static_assert(ROWS % (8 * NW) == 0 && BM % (8 * NW) == 0, "whole loads");
    static_assert(SLOTS % RING == 0 && RING <= WB && LPT <= SLOTS, "slots");
    __shared__ u32x4 lds[2 * STAGE];

    GemmProblem P;
    int tile, zero_n;
    int32_t* zero_ptr;
    if (!gemm_pick_tile(g, tile, P, zero_n, zero_ptr)) return;
    const int local = tile - P.tile_begin;
    const int band_tiles = 8 * P.tiles_n;
    const int band = local / band_tiles, rem = local - band * band_tiles;
    const int band_rows = min(8, P.tiles_m - band * 8);
    const int tn = rem / band_rows, tm = band * 8 + rem % band_rows;
    const int m0 = tm * BM, n0 = tn * GG_OUT;
    const int Mp = P.Mp, F = P.N, r = P.K1;
    const int nk0 = P.K0 / 64, nkt = nk0 + (r + 63) / 64;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int wm = (wave >> 1) * (MI * 32), wn = (wave & 1) * (GG_BN / 2);

    // row of W behind row j of the tile: blocks of 16 value rows and the 16 gate rows of the same output columns take turns
    auto wrow = [&](int j) { return min(n0 + (j >> 5) * 16 + (j & 15), F - 1) + ((j >> 4) & 1) * F; };
    // load j of wavefront w fills block j * NW + w of a stage: the rows of x first, then those of W
    uint32_t off[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int row = (j * NW + wave) * 8 + (lane >> 3), c = swz<8>(row, lane & 7);
        if (j < JP) off[j] = (uint32_t)(((min(m0 + row, Mp - 1) - m0) * P.ldp0 + c * 8) * 2);
        else off[j] = (uint32_t)((wrow(row - BM) * P.ldq0 + c * 8) * 2);
    }
    const uint16_t* const pb0 = P.p0 + (int64_t)m0 * P.ldp0;
    const uint32_t wave_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds + (uint32_t)wave * 1024;
    auto load = [&](int t, int stg, int j) {
        dma16_so<false>((j < JP ? pb0 : P.q0) + t * 64, off[j], wave_base + (uint32_t)(stg * (STAGE * 16) + j * (NW * 1024)));
    };
    // tile of the adapter's segment: t [M, r] and B [2F, r]; chunks past r read zeros.  (From a lane number that the compiler
    // does not know: it would form the addresses ahead of the main loop and spill there.)
    auto load1 = [&](int t, int stg, int j, int ln) {
        const int row = (j * NW + wave) * 8 + (ln >> 3), c = swz<8>(row, ln & 7), k = (t - nk0) * 64 + c * 8;
        const uint16_t* src = j < JP ? P.p1 + (int64_t)min(m0 + row, Mp - 1) * P.ldp1 : P.q1 + (int64_t)wrow(row - BM) * P.ldq1;
        dma16<false>(k < r ? reinterpret_cast<const void*>(src + k) : reinterpret_cast<const void*>(g_gemm_zeros),
                     wave_base + (uint32_t)(stg * (STAGE * 16) + j * (NW * 1024)));
    };
    auto issue = [&](int t, int stg) {
        if (t < nk0) {
#pragma unroll
            for (int j = 0; j < LPT; ++j) load(t, stg, j);
        } else {
            int ln = lane;
            asm volatile("" : "+v"(ln));
#pragma unroll
            for (int j = 0; j < LPT; ++j) load1(t, stg, j, ln);
        }
    };

    f32x4 acc[XB][WB];
#pragma unroll
    for (int mi = 0; mi < XB; ++mi)
#pragma unroll
        for (int ni = 0; ni < WB; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the x blocks of both k-steps, and a ring of W blocks: slot s multiplies W block s % WB in k-step s / WB out of wf[s % RING],
    // which is then refilled for slot s + RING, over the edge of two tiles too
    bf16x8 xf[2][XB], wf[RING];
    const int lrow = l16 * 8, lsw = (l16 >> 1) & 7;
    auto frag = [&](int st, int ks) { return lds + (st * STAGE + lrow + ((ks * 4 + quad) ^ lsw)); };
    auto fetch_x = [&](int st, int ks) {
        const u32x4* const sx = frag(st, ks) + wm * 8;
#pragma unroll
        for (int mi = 0; mi < XB; ++mi) xf[ks][mi] = __builtin_bit_cast(bf16x8, sx[mi * 128]);
    };
    auto fetch_w = [&](int st, int s) { wf[s % RING] = __builtin_bit_cast(bf16x8, (frag(st, s / WB) + (BM + wn) * 8)[(s % WB) * 128]); };
    auto multiply = [&](int s) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < XB; ++mi)
            acc[mi][s % WB] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s % RING], xf[s / WB][mi], acc[mi][s % WB], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto no_load = [](int) {};
    // all slots of a tile but the last RING, loads [j0, LPT) of another dealt behind them
    auto head = [&](int st, auto ld, int j0) {
#pragma unroll
        for (int s = 0; s < SLOTS - RING; ++s) {
            if (s == 0) fetch_x(st, 1);
            multiply(s);
            if (j0 + s < LPT) ld(j0 + s);
            fetch_w(st, s + RING);
        }
    };
    // the last RING slots of a tile, whose operands are in registers, while the first of the next are read
    auto edge = [&](int sn, auto ld) {
        fetch_x(sn, 0);
#pragma unroll
        for (int i = 0; i < RING; ++i) {
            multiply(SLOTS - RING + i);
            if (i < LPT) ld(i);
            fetch_w(sn, i);
        }
    };

    issue(0, 0);
    if (nkt > 1) issue(1, 1);
    if (nkt > 1) wait_vmcnt<LPT>();
    else wait_vmcnt<0>();
    __syncthreads();
    fetch_x(0, 0);
#pragma unroll
    for (int s = 0; s < RING; ++s) fetch_w(0, s);
    head(0, no_load, LPT);

    // a step: the edge between tiles t and t+1, before tile t's last slots (whose operands are in
    // registers); the stage of tile t takes tile t+2
    int t = 0;
#pragma unroll 1
    for (; t + 2 < nk0; ++t) {
        const int st = t & 1, sn = st ^ 1;
        wait_vmcnt<0>();
        __syncthreads();
        auto ld = [&](int j) { load(t + 2, st, j); };
        edge(sn, ld);
        head(sn, ld, RING);
    }
#pragma unroll 1
    for (; t + 1 < nkt; ++t) {
        const int st = t & 1, sn = st ^ 1;
        wait_vmcnt<0>();
        __syncthreads();
        if (t + 2 < nkt) issue(t + 2, st);
        edge(sn, no_load);
        head(sn, no_load, LPT);
    }
#pragma unroll
    for (int s = SLOTS - RING; s < SLOTS; ++s) multiply(s);

    // ---- bias, GEGLU, store
    const float alpha = P.alpha;
    const uint16_t* const bias = P.bias;
#pragma unroll
    for (int p = 0; p < WB / 2; ++p) {
        const int n = n0 + (wn >> 1) + p * 16 + quad * 4;
        if (n >= F) continue;       // F is a multiple of 8
        u32x2 b0 = {0u, 0u}, b1 = {0u, 0u};
        if (bias) {
            b0 = *reinterpret_cast<const u32x2*>(bias + n);
            b1 = *reinterpret_cast<const u32x2*>(bias + F + n);
        }
#pragma unroll
        for (int mi = 0; mi < XB; ++mi) {
            const int m = m0 + wm + mi * 16 + l16;
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float bv = e & 1 ? bf16hi_to_f32(b0[e >> 1]) : bf16lo_to_f32(b0[e >> 1]);
                const float bg = e & 1 ? bf16hi_to_f32(b1[e >> 1]) : bf16lo_to_f32(b1[e >> 1]);
                o[e] = (__bf16)((alpha * acc[mi][2 * p][e] + bv) * gelu_erf(alpha * acc[mi][2 * p + 1][e] + bg));
            }
            if (m < Mp) *reinterpret_cast<bf16x4*>(static_cast<uint16_t*>(P.y) + (int64_t)m * P.ldy + n) = o;
        }
    }
}

// ---- the adapter's down-projection in front of it: 32 rows x 64 columns per workgroup, so that a few
// thousand rows still reach every CU; two column wavefronts' worth of K halves.  Bound by latency (one
// load round trip per 640 of K): two stages of 320 in flight, no tile of any other kind waits for it.
constexpr int DN_BM = 32, DN_BN = 64, DN_KB = 5;               // rows, columns, 64 deep blocks per stage
__global__ __launch_bounds__(512, 2) void down_kernel(const uint16_t* __restrict__ x, int64_t ldx, const uint16_t* __restrict__ A, float scale,
                                                      uint16_t* __restrict__ t, int M, int K, int r) {
    constexpr int ROWS = DN_BM + DN_BN, BLK = ROWS * 8;        // 16-byte chunks of a 64 deep block
    constexpr int NL = ROWS / 8 * DN_KB, LPT = (NL + 7) / 8;   // 1 KB loads of a stage, and per wavefront
    constexpr int STAGE = BLK * DN_KB;
    __shared__ u32x4 lds[2 * STAGE];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int m0 = blockIdx.x * DN_BM, c0 = blockIdx.y * DN_BN;
    const int nb = K / 64, ns = (nb + DN_KB - 1) / DN_KB;
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    auto issue = [&](int s, int stg) {
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const int l = min(j * 8 + wave, NL - 1);           // the last load once more where 8 does not divide them
            const int kb = l / (ROWS / 8), row = (l % (ROWS / 8)) * 8 + (lane >> 3);
            const int k = min(s * DN_KB + kb, nb - 1) * 64 + swz<8>(row, lane & 7) * 8;
            const uint16_t* const src = row < DN_BM ? x + (int64_t)min(m0 + row, M - 1) * ldx : A + (int64_t)min(c0 + row - DN_BM, r - 1) * K;
            dma16<false>(src + k, base + (uint32_t)(stg * (STAGE * 16) + l * 1024));
        }
    };
    issue(0, 0);
    if (ns > 1) issue(1, 1);
    const int col = (wave & 3) * 16, wk = wave >> 2;
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const int lsw = (l16 >> 1) & 7;
#pragma unroll 1
    for (int s = 0; s < ns; ++s) {
        if (s + 1 < ns) wait_vmcnt<LPT>();
        else wait_vmcnt<0>();
        __syncthreads();
#pragma unroll
        for (int kb = 0; kb < DN_KB; ++kb)
            if (s * DN_KB + kb < nb) {
                const u32x4* const b = lds + (s & 1) * STAGE + kb * BLK + l16 * 8 + ((wk * 4 + quad) ^ lsw);
                const bf16x8 a = __builtin_bit_cast(bf16x8, b[(DN_BM + col) * 8]);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, b[i * 128]), acc[i], 0, 0, 0);
            }
        __syncthreads();
        if (s + 2 < ns) issue(s + 2, s & 1);
    }
    f32x4* const ex = reinterpret_cast<f32x4*>(lds);
    if (wk == 1) {
        ex[((wave & 3) * 2 + 0) * 64 + lane] = acc[0];
        ex[((wave & 3) * 2 + 1) * 64 + lane] = acc[1];
    }
    __syncthreads();
    if (wk == 0) {
        const int c = c0 + col + quad * 4;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const f32x4 v = acc[i] + ex[(wave * 2 + i) * 64 + lane];
            const int m = m0 + i * 16 + l16;
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (__bf16)(v[e] * scale);
            if (m < M && c < r) *reinterpret_cast<bf16x4*>(t + (int64_t)m * r + c) = o;    // r is a multiple of 8
        }
    }
}

// ---- the same for few rows or ranks: BM rows x 16 columns per workgroup.  Bound by latency: a wavefront loads 64 deep
// blocks of both operands, every eighth, into LDS of its own, all of them at once up to K = 1536 (2048 with 16 rows), and the workgroup
// meets once, to add up eight partial sums.
template <int BM>
__global__ __launch_bounds__(512, 2) void down16_kernel(const uint16_t* __restrict__ x, int64_t ldx, const uint16_t* __restrict__ A, float scale,
                                                        uint16_t* __restrict__ t, int M, int K, int r) {
    constexpr int ROWS = BM + 16, BLK = ROWS * 8, NL = ROWS / 8;    // 16-byte chunks of a block, its 1 KB loads
    constexpr int DEPTH = BM == 32 ? 3 : 4, MI = BM / 16;           // blocks of a wavefront in flight
    __shared__ u32x4 lds[8 * DEPTH * BLK];
    static_assert(sizeof(lds) <= 160 * 1024 && MI * 64 <= DEPTH * BLK, "LDS");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int m0 = blockIdx.x * BM, c0 = blockIdx.y * 16;
    const int mine = (K / 64 - wave + 7) / 8;
    u32x4* const own = lds + wave * (DEPTH * BLK);
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds + (uint32_t)wave * (DEPTH * BLK * 16);
    const uint16_t* src[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int row = j * 8 + (lane >> 3);
        src[j] = (row < BM ? x + (int64_t)min(m0 + row, M - 1) * ldx : A + (int64_t)min(c0 + row - BM, r - 1) * K) + wave * 64 + swz<8>(row, lane & 7) * 8;
    }
    auto issue = [&](int i, int slot) {
#pragma unroll
        for (int j = 0; j < NL; ++j) dma16<false>(src[j] + i * 512, base + (uint32_t)(slot * (BLK * 16) + j * 1024));
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (d < mine) issue(d, d);
    f32x4 acc[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) acc[mi] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int lsw = (l16 >> 1) & 7;
    int slot = 0;
#pragma unroll 1
    for (int i = 0; i < mine; ++i) {
        const int newer = mine - 1 - i;         // blocks that may stay in flight
        if (DEPTH >= 4 && newer >= 3) wait_vmcnt<3 * NL>();
        else if (newer >= 2) wait_vmcnt<2 * NL>();
        else if (newer == 1) wait_vmcnt<NL>();
        else wait_vmcnt<0>();
        bf16x8 a[2], xf[2][MI];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const u32x4* const b = own + slot * BLK + l16 * 8 + ((kk * 4 + quad) ^ lsw);
            a[kk] = __builtin_bit_cast(bf16x8, b[BM * 8]);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) xf[kk][mi] = __builtin_bit_cast(bf16x8, b[mi * 128]);
        }
        // the block is in registers: its place takes another
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (i + DEPTH < mine) issue(i + DEPTH, slot);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) acc[mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk], xf[kk][mi], acc[mi], 0, 0, 0);
        slot = slot + 1 == DEPTH ? 0 : slot + 1;
    }
    f32x4* const part = reinterpret_cast<f32x4*>(own);
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) part[mi * 64 + lane] = acc[mi];
    __syncthreads();
    if (wave < MI) {
        const f32x4* const p = reinterpret_cast<const f32x4*>(lds) + wave * 64 + lane;
        f32x4 v = p[0];
#pragma unroll
        for (int w = 1; w < 8; ++w) v += p[w * (DEPTH * BLK)];
        const int m = m0 + wave * 16 + l16, c = c0 + quad * 4;
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)(v[e] * scale);
        if (m < M && c < r) *reinterpret_cast<bf16x4*>(t + (int64_t)m * r + c) = o;    // r is a multiple of 8
    }
}
// 16 columns a workgroup while all of them are one round, and at rank 16 and less, where 32x64 loads rows of A that it has no use for; 16 rows
// where that is one round, too.  us a launch in the stacks, 32x64 / here: 2048x1280 + 64 6.62 / 4.86 (64 workgroups and 256).  With the wide tiles behind it,
// weights in L2, 32x64 / 32x16 / 16x16: 988x5120x1280 + 64 35.3 / 32.8 / 32.6, 1800x2560x640 + 32 22.9 / 21.4 / 21.1; 32x64 / 32x16: 2048x5120x1280 + 64
// 53.1 / 50.6, 8192x1280x320 + 16 26.1 / 25.5, 16384x2560x640 + 16 124.5 / 122.9.  In more than a round every column tile reads the rows
// again: 3952x2560x640 + 64 35.4 / 36.0, 8192x2560x640 + 32 64.8 / 65.7, + 64 65.9 / 69.6.
int launch_down(const uint16_t* x, int64_t ldx, const uint16_t* A, float scale, uint16_t* t, int M, int K, int r, hipStream_t stream) {
    const int n16 = (r + 15) / 16;
    const bool narrow = n16 == 1 || (M + 31) / 32 * n16 <= 256, low = narrow && (M + 15) / 16 * n16 <= 256;
    const int rows = low ? 16 : DN_BM, cols = narrow ? 16 : DN_BN;
    if (SD_DRY_RUN("down%s; ", dry_detail(narrow ? ", %d rows by 16" : ", %d rows by 64", rows))) return SD_OK;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((M + rows - 1) / rows, (r + cols - 1) / cols), dim3(512), 0, stream, x, ldx, A, scale, t, M, K, r);
    };
    if (low) launch(down16_kernel<16>);
    else if (narrow) launch(down16_kernel<32>);
    else launch(down_kernel);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

template <int MI>
static int launch_geglu_mi(GemmGroup& g, hipStream_t stream) {
    GemmProblem& P = g.p[0];
    P.tiles_m = (P.Mp + MI * 128 - 1) / (MI * 128);
    P.tiles_n = (P.N + GG_OUT - 1) / GG_OUT;
    P.tile_begin = g.first_tile[0] = 0;
    g.n_lead = 0;
    g.total_tiles = P.tiles_m * P.tiles_n;
    if (SD_DRY_RUN("geglu %dx160; ", MI * 128)) return SD_OK;
    hipLaunchKernelGGL((gemm_geglu_kernel<MI>), dim3((g.total_tiles + 7) & ~7), dim3(512), 0, stream, g);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}
// Which tiles.  Up to four 64x64 tiles per CU, that many workgroups of the general kernel in one round: 64x64 (three
// ring stages while there are at most two per CU and the K loop is not short), 128x64 from three on.  Beyond that the
// estimate, us, fitted to 600 launches of 154 to 16384 rows and C = 320 to 2048 before 16x16x32 MFMAs and 16 columns a workgroup in the
// down-projection: rounds of workgroups over 256 CUs (128x64: over two per CU), each with a fixed part and one per 64 deep step; the wide tiles' down-projection is a
// launch of its own where the general kernel hides it.  With the kernels as they are, over 120 launches of 154 to 16384 rows, C = 320 to 1280 and ranks 0 to 128 behind a LayerNorm: 0.4 %
// slower than the best of the six in the mean, one in thirty by more than 3 %, none by more than 8.  Without a LayerNorm in front (no launch of the transformer block), 50 launches: 4 % in the mean,
// one in four by more than 3 %, the worst by 35 (1032x2560x640 + 64 23.3, 17.3 with 128x64).  us with the LayerNorm, 64x64 with three stages / 64x64 / 128x64 / 256x128 / wide 256 /
// wide 128: 2048x1280x320 + 8 21.2 17.1 17.6 21.7 24.5 17.4; 988x5120x1280 39.7 40.0 43.1 42.0 41.1 32.4; 7904x2560x640 80.7 79.2 71.3 79.0 63.4 71.4; 7904x4096x2048 316 315 270
// 241 252 268; 8192x2560x640 + 64 89.3 88.0 83.0 82.2 73.0 82.3.
GegluTiles geglu_tiles(int M, int F, int K, int r, bool wide_ok) {
    const int k_steps = K / 64, steps = k_steps + (r + 63) / 64;
    auto tiles = [&](int rows, int cols) { return (long)((M + rows - 1) / rows) * ((F + cols - 1) / cols); };
    const long t64 = tiles(64, 64);
    if (t64 <= 256) return k_steps <= 5 && r > 0 ? GEGLU_64x64 : GEGLU_64x64_3STAGES;
    if (t64 <= 2 * 256) return k_steps <= 10 ? GEGLU_64x64 : GEGLU_64x64_3STAGES;
    if (t64 <= 3 * 256) return GEGLU_64x64;
    if (t64 <= 4 * 256) return GEGLU_128x64;
    auto us = [&](long n, int slots, double fixed, double per_step) { return (double)((n + slots - 1) / slots) * (fixed + per_step * steps); };
    const double down = r > 0 ? 3.5 + 1.7 * (double)((M + 31) / 32) * ((r + 63) / 64) / 256 : 0.0;
    GegluTiles best = GEGLU_128x64;
    double least = us(tiles(128, 64), 512, 3.8, 0.90);
    auto consider = [&](GegluTiles t, double v) {
        if (v < least) { least = v; best = t; }
    };
    consider(GEGLU_256x128, us(tiles(256, 128), 256, 7.3, 1.73));
    if (wide_ok) {
        consider(GEGLU_WIDE_256x160, us(tiles(256, GG_OUT), 256, 10.4, 1.75) + down);
        consider(GEGLU_WIDE_128x160, us(tiles(128, GG_OUT), 256, 6.0, 1.08) + down);
    }
    return best;
}
bool gemm_geglu_takes(const GemmProblem& P) {
    return P.geglu_F == P.N && P.N > 0 && P.Mp > 0 && P.K0 % 64 == 0 && P.N % 8 == 0 && P.ldy % 8 == 0 && !P.y_f32 && !P.res && !P.bias_on_rows && aligned16(P.bias) && aligned16(P.y) &&
           P.ldp0 * 512 < (1ll << 31) && P.ldq0 * 4 * P.N < (1ll << 32) && geglu_tiles(P.Mp, P.N, P.K0, P.K1, true) >= GEGLU_WIDE_256x160;
}
int launch_gemm_geglu(GemmGroup& g, hipStream_t stream) {
    const GemmProblem& P = g.p[0];
    return geglu_tiles(P.Mp, P.N, P.K0, P.K1, true) == GEGLU_WIDE_256x160 ? launch_geglu_mi<2>(g, stream) : launch_geglu_mi<1>(g, stream);
}

}  // namespace sd
