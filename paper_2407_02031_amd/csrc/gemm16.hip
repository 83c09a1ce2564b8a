// Projections whose tiles cover the chip in whole rounds: bf16 MFMA GEMM with 16-granular tiles
// and the adapter's down-projection computed inside the tile.
//
// What bounds it: at the block's sizes one projection is one or two tiles per CU, so its time is
// that of the most loaded CU: launch, first loads, the K loop at the rate a CU takes operands in
// from L2 (100-125 GB/s) or multiplies them, and the stores.  Tiles of 128x160, 64x160 and 64x80 give
// all 256 CUs the same work where powers of two do not (8192x640 and 2048x1280 are 256 tiles of
// 128x160 and 64x160).
//
// A tile's wavefronts split its K as well as its rows and columns (WGK groups each multiply every
// WGK-th 32 deep k-step of a 64 deep stage): larger wavefront tiles, so fewer LDS reads per MFMA,
// with two wavefronts per SIMD all the same.  The groups' sums are added through LDS at the end.
//
// LoRA: the tile carries the r rows of A as further columns of its product, t = x A^T, and when
// the K loop is done adds (scale t) B^T out of LDS.  Every column tile of a row block repeats
// that, which is cheaper at these sizes than a producer tile, its stores and the wait for them;
// t is rounded to bf16 as if it had been stored.
//
// The MFMA is issued with the weight rows as its first operand: a lane then holds four
// consecutive output columns of one row, and bias, residual and store need no staging.
#include "gemm_dma.hpp"

namespace sd {

// DEPTH: ring stages of a tile of which 160 KB hold six or more
template <int BM, int BN, int WGM, int WGN, int WGK, int NRB, int DEPTH>
struct Tile16 {
    static constexpr int NW = WGM * WGN * WGK;
    static constexpr int MI = BM / WGM / 16, NI = BN / WGN / 16;   // 16x16 blocks of a wavefront
    static constexpr int RN = NRB * 16 * WGN;                      // rows of A in a stage
    static constexpr int ROWS = BM + BN + RN;
    static constexpr int NBLK = ROWS / 8;                          // 1 KB blocks (8 rows of 128 bytes) of a stage
    static constexpr int LPT = (NBLK + NW - 1) / NW;               // loads per wavefront and stage
    static constexpr int STAGE_CH = ROWS * 8;                      // 16-byte chunks of a stage
    static constexpr int FIT = 160 * 1024 / (ROWS * 128);
    static constexpr int STAGES = FIT >= 6 ? DEPTH : FIT;
    static constexpr int EXCH = WGK > 1 ? NW * (MI / 2) * NI * 64 : 0;   // chunks of the exchange of the groups' sums
    static constexpr int LDS_CH = STAGES * STAGE_CH > EXCH ? STAGES * STAGE_CH : EXCH;
    static_assert(WGK == 1 || WGK == 2, "a stage has two 32 deep k-steps");
    static_assert(STAGES >= 3 && STAGES <= 5, "ring");
    static_assert(WGK == 1 || MI % 2 == 0, "the groups share the epilogue by row blocks");
    static_assert(BM * RN * 4 <= STAGE_CH * 16, "the exchange of t fits a stage");
};

template <int V> struct IntC { static constexpr int v = V; };
constexpr int RES_NONE = 0, RES_BF16 = 1, RES_F32 = 2;

template <int BM, int BN, int WGM, int WGN, int WGK, int NRB, int RES, int DEPTH>
__global__ __launch_bounds__(64 * WGM * WGN * WGK, 2) void gemm16_kernel(const GemmGroup g) {
    using T = Tile16<BM, BN, WGM, WGN, WGK, NRB, DEPTH>;
    constexpr int NW = T::NW, MI = T::MI, NI = T::NI, RN = T::RN, LPT = T::LPT, STAGES = T::STAGES, STAGE = T::STAGE_CH, NBLK = T::NBLK;
    constexpr int PH = 2 / WGK;             // k-steps of a stage that this wavefront multiplies
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
    const int Mp = P.Mp, N = P.N, r = NRB ? P.K1 : 0;
    const int nk0 = P.K0 / 64, nkt = nk0 + (r ? 1 : 0);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int wk = wave / (WGM * WGN), wmn = wave % (WGM * WGN);
    const int wm = (wmn / WGN) * (BM / WGM), wn = (wmn % WGN) * (BN / WGN), wr = (wmn % WGN) * (NRB * 16);

    // ---- loader.  Load j of wavefront w fills 1 KB block j * NW + w of a stage (x rows, W rows, A rows);
    // where NW does not divide the blocks, the last wavefronts load the last block once more.
    // (every wavefront-uniform choice is a select of scalars: as branches they cost more than the first loads' latency)
    uint32_t off[LPT];            // byte offset of this lane's chunk from its operand's first row
    uint32_t offb[LPT];           // ... in the tile of B (P.q1), or past what it holds: NONE
    const char* base[LPT];
    int dst[LPT];
    constexpr uint32_t NONE = 0xffffffffu;
    const char* const xbase = reinterpret_cast<const char*>(P.p0 + (int64_t)m0 * P.ldp0);
    const char* const wbase = reinterpret_cast<const char*>(P.q0 + (int64_t)n0 * P.ldq0);
    const char* const abase = reinterpret_cast<const char*>(r ? P.p1 : P.q0);   // (a projection without adapter in a launch that has some: rows of W, and nothing done with the product)
    const int xld = (int)P.ldp0 * 2, wld = (int)P.ldq0 * 2, ald = r ? (int)P.ldp1 * 2 : 0, bld = (int)P.ldq1 * 2;
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int blk = min(j * NW + wave, NBLK - 1);
        dst[j] = blk * 1024;
        const int row = blk * 8 + (lane >> 3);
        const int c16 = swz<8>(row, lane & 7) * 16;
        const bool isx = blk < BM / 8, isa = NRB && blk >= (BM + BN) / 8;
        const int first = isx ? 0 : isa ? BM + BN : BM;
        const int last = isx ? Mp - 1 - m0 : isa ? (r ? r - 1 : 0) : N - 1 - n0;
        const int ld = isx ? xld : isa ? ald : wld;
        base[j] = isx ? xbase : isa ? abase : wbase;
        const int k = min(row - first, last);
        off[j] = (uint32_t)(k * ld + c16);
        offb[j] = NRB && !isx && !isa && c16 < 2 * r ? (uint32_t)(k * bld + c16) : NONE;
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    auto load = [&](int t, int stg, int j) {
        dma16_so<false>(base[j] + (int64_t)t * 128, off[j], lds_base + (uint32_t)(stg * (STAGE * 16) + dst[j]));
    };
    // the tile of B: every lane has an address of its own, chunks past its r columns (and the other
    // operands' blocks) read zeros; as many loads as any stage, so that the wait counts hold
    auto load_b = [&](int stg, int j) {
        const char* src = reinterpret_cast<const char*>(P.q1 + (int64_t)n0 * P.ldq1) + offb[j];
        src = offb[j] != NONE ? src : reinterpret_cast<const char*>(g_gemm_zeros);
        dma16<false>(src, lds_base + (uint32_t)(stg * (STAGE * 16) + dst[j]));
    };
    auto issue = [&](int t, int stg) {
        if (NRB == 0 || t < nk0) {
#pragma unroll
            for (int j = 0; j < LPT; ++j) load(t, stg, j);
        } else {
#pragma unroll
            for (int j = 0; j < LPT; ++j) load_b(stg, j);
        }
    };

    f32x4 acc[MI][NI], acct[MI][NRB ? NRB : 1];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ri = 0; ri < NRB; ++ri) acct[mi][ri] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 xf[2][MI], wf[2][NI], rf[2][NRB ? NRB : 1];
    // rows that are 16 apart share the swizzle: one LDS address per k-step, the rest are offsets
    const int lrow = l16 * 8, lsw = (l16 >> 1) & 7;
    auto frag = [&](int st, int kk) { return lds + (st * STAGE + lrow + ((kk * 4 + quad) ^ lsw)); };
    auto fetch_x = [&](int st, int kk, int fs) {
        const u32x4* const sx = frag(st, kk) + wm * 8;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) xf[fs][mi] = __builtin_bit_cast(bf16x8, sx[mi * 128]);
    };
    auto fetch_w = [&](int st, int kk, int fs) {
        const u32x4* const sw = frag(st, kk) + (BM + wn) * 8;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) wf[fs][ni] = __builtin_bit_cast(bf16x8, sw[ni * 128]);
    };
    auto fetch = [&](int st, int kk, int fs) {
        const u32x4* const sr = frag(st, kk) + (BM + BN + wr) * 8;
        fetch_x(st, kk, fs);
        fetch_w(st, kk, fs);
#pragma unroll
        for (int ri = 0; ri < NRB; ++ri) rf[fs][ri] = __builtin_bit_cast(bf16x8, sr[ri * 128]);
    };
    // one k-step, loads [j0, j1) dealt between its MFMAs
    auto multiply = [&](int fs, bool down, auto ld, int j0, int j1) {
        constexpr int NT = NI + NRB;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < MI * NT; ++i) {
            const int mi = i % MI, ni = i / MI;
            if (ni < NI)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[fs][ni], xf[fs][mi], acc[mi][ni], 0, 0, 0);
            else if (down)
                acct[mi][ni - NI] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rf[fs][ni - NI], xf[fs][mi], acct[mi][ni - NI], 0, 0, 0);
            const int a = j0 + (j1 - j0) * i / (MI * NT), b = j0 + (j1 - j0) * (i + 1) / (MI * NT);
            if (a < b) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = a; j < b; ++j) ld(j);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto no_load = [](int) {};
    // ---- what the epilogue adds, requested when the first stage has landed: as long as one of the first STAGES is waited
    // for, these NEXTRA loads may stay in flight too (loads retire in order).  Every lane loads, rows and columns past the end their
    // last ones, and the compiler does not see which columns those are: equal addresses (no bias) would be one load, and the waits, which
    // count NEXTRA, would let a stage's own loads pass.  (Requested at the last MFMAs, as before, a launch that is one round of
    // tiles has nothing to hide them behind.  With the branch-free prologue and the straight-line epilogue below, operands from
    // HBM: 8192x640x640 + 64 with an fp32 residual 24.2 -> 23.4 us, 1000x640x640 + 32 9.2 -> 8.2, 512x320x320 + 8 6.6 -> 6.0.)
    constexpr int ME = WGK == 2 ? MI / 2 : MI;   // row blocks this wavefront finishes
    const int mfirst = WGK == 2 ? wk * ME : 0;
    const int mrow = m0 + wm + mfirst * 16 + l16, ncol = n0 + wn + quad * 4;
    constexpr int NEXTRA = NI + (RES ? ME * NI : 0);
    f32x4 resf[RES == RES_F32 ? ME : 1][NI];
    u32x2 resb[RES == RES_BF16 ? ME : 1][NI], bias[NI];
    auto load_extra = [&]() {
        const uint16_t* const bp = P.bias ? P.bias : reinterpret_cast<const uint16_t*>(g_gemm_zeros);
        int col[NI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            col[ni] = min(ncol + ni * 16, N - 4);
            uint32_t at = P.bias ? col[ni] : 0;
            asm volatile("" : "+v"(at));
            bias[ni] = *as_global(reinterpret_cast<const u32x2*>(bp + at));
        }
#pragma unroll
        for (int mi = 0; mi < (RES ? ME : 0); ++mi) {
            int64_t row = (int64_t)min(mrow + mi * 16, Mp - 1) * P.ldr;
            asm volatile("" : "+v"(row));
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int64_t at = row + col[ni];
                if (RES == RES_F32) resf[mi][ni] = *as_global(reinterpret_cast<const f32x4*>(static_cast<const float*>(P.res) + at));
                else resb[mi][ni] = *as_global(reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(P.res) + at));
            }
        }
    };
    // tiles newer than the one waited for, which may stay in flight, and the loads above with them
    auto wait_more = [&](int newer, auto extra) {
        constexpr int E = decltype(extra)::v;
        if (STAGES >= 5 && newer >= 4) wait_vmcnt<4 * LPT + E>();
        else if (STAGES >= 4 && newer >= 3) wait_vmcnt<3 * LPT + E>();
        else if (newer >= 2) wait_vmcnt<2 * LPT + E>();
        else if (newer >= 1) wait_vmcnt<LPT + E>();
        else wait_vmcnt<E>();
    };
    auto wait_tiles = [&](int newer, bool first) {      // first: the tile is one of the first STAGES
        if (first) wait_more(newer, IntC<NEXTRA>());
        else wait_more(newer, IntC<0>());
    };

    // ---- prologue
#pragma unroll
    for (int d = 0; d < STAGES; ++d)
        if (d < nkt) issue(d, d);
    wait_tiles(min(nkt - 1, STAGES - 1), false);
    __syncthreads();
    fetch(0, wk, 0);
    load_extra();
    if (PH == 2) {
        fetch(0, 1, 1);
        multiply(0, true, no_load, 0, 0);
    }

    // ---- K loop.  A step's edge lies before the MFMAs of tile t's last k-step, whose fragments are in
    // registers: when this wavefront's loads of tile t+1 have landed, one barrier says that tile t+1
    // is whole and the stage of tile t free; that is refilled with tile t+STAGES, its loads dealt over
    // the step's MFMAs, and the first fragments of tile t+1 are read meanwhile.  With one k-step per
    // stage the two fragment sets take turns from step to step.
    // Steps that may wait for one of the first STAGES tiles have a loop of their own: asked in every step, that choice took 23 ns of
    // 245 with four stages and 11 with three (80 steps, 73x1280x5120 with an fp32 residual 19.7 us, 17.9 without; 154x1280x2048 + 8 11.5 / 10.9).
    constexpr int TAIL = 0, FULL = 1, FULL_FIRST = 2;
    int st = 0, t = 0;
    auto step = [&](auto par, auto full) {
        constexpr int FS = PH == 2 ? 1 : decltype(par)::v;
        if (decltype(full)::v) wait_tiles(STAGES - 2, decltype(full)::v == FULL_FIRST && t + 1 < STAGES);
        else wait_tiles(min(nkt - 2 - t, STAGES - 2), t + 1 < STAGES);
        __syncthreads();
        const int sn = st + 1 == STAGES ? 0 : st + 1;
        fetch(sn, wk, FS ^ 1);
        if (decltype(full)::v) {
            auto ld = [&](int j) { load(t + STAGES, st, j); };
            multiply(FS, true, ld, 0, LPT / PH);
            if (PH == 2) {
                fetch(sn, 1, 1);
                multiply(0, true, ld, LPT / PH, LPT);
            }
        } else {
            if (t + STAGES < nkt) issue(t + STAGES, st);
            multiply(FS, true, no_load, 0, 0);
            if (PH == 2) {
                fetch(sn, 1, 1);
                multiply(0, true, no_load, 0, 0);
            }
        }
        st = sn;
        ++t;
    };
    // (an odd number of steps: one ahead of the pairs, and its fragments moved to the first set)
    if ((nk0 - 1) & 1) {
        step(IntC<0>(), IntC<TAIL>());
        if (PH == 1) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) xf[0][mi] = xf[1][mi];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) wf[0][ni] = wf[1][ni];
#pragma unroll
            for (int ri = 0; ri < NRB; ++ri) rf[0][ri] = rf[1][ri];
        }
    }
#pragma unroll 1
    while (t + 1 < STAGES && t + 1 + STAGES < nk0) {
        step(IntC<0>(), IntC<FULL_FIRST>());
        step(IntC<1>(), IntC<FULL_FIRST>());
    }
#pragma unroll 1
    while (t + 1 + STAGES < nk0) {
        step(IntC<0>(), IntC<FULL>());
        step(IntC<1>(), IntC<FULL>());
    }
#pragma unroll 1
    while (t + 1 < nk0) {
        step(IntC<0>(), IntC<TAIL>());
        step(IntC<1>(), IntC<TAIL>());
    }

    multiply(PH == 2 ? 1 : 0, true, no_load, 0, 0);

    // ---- adapter: t = x A^T is whole (over the K groups) after this, rounded to bf16, and becomes the
    // x part of the stage that holds B
    if (NRB && r) {
        wait_vmcnt<0>();
        __syncthreads();                    // the tile of B has landed; every fragment of the last tile is in registers
        const int sb = st + 1 == STAGES ? 0 : st + 1;
        const bool both = PH == 2 && r > 32;                                 // its second k-step holds columns of the adapter too
        fetch_w(sb, wk, 0);
        if (both) fetch_w(sb, 1, 1);
        f32x4* const xch = reinterpret_cast<f32x4*>(lds + st * STAGE) + wmn * (MI * NRB * 64) + lane;
        if (WGK == 2) {
            if (wk == 1)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ri = 0; ri < NRB; ++ri) xch[(mi * NRB + ri) * 64] = acct[mi][ri];
            __syncthreads();
        }
        if (wk == 0) {
            uint16_t* const tb = reinterpret_cast<uint16_t*>(lds + sb * STAGE);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ri = 0; ri < NRB; ++ri) {
                    f32x4 v = acct[mi][ri];
                    if (WGK == 2) v += xch[(mi * NRB + ri) * 64];
                    const int row = wm + mi * 16 + l16, col = wr + ri * 16 + quad * 4;
                    bf16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = (__bf16)(col + e < r ? v[e] * P.t_scale : 0.f);
                    *reinterpret_cast<bf16x4*>(tb + row * 64 + swz<8>(row, col >> 3) * 8 + (col & 4)) = o;
                }
        }
        // (a rank of at most RN: what lies between its columns and the 64 of the stage was loaded as zeros)
        __syncthreads();
        fetch_x(sb, wk, 0);
        if (both) fetch_x(sb, 1, 1);
        multiply(0, false, no_load, 0, 0);
        if (both) multiply(1, false, no_load, 0, 0);
    }

    // ---- sums of the K groups: each gives the other the half of the row blocks it does not finish
    f32x4 fin[ME][NI];
    if (WGK == 2) {
        __syncthreads();
        f32x4* const ex = reinterpret_cast<f32x4*>(lds) + lane;
        constexpr int PER = ME * NI * 64;
#pragma unroll
        for (int mi = 0; mi < ME; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                ex[wave * PER + (mi * NI + ni) * 64] = wk ? acc[mi][ni] : acc[ME + mi][ni];
                fin[mi][ni] = wk ? acc[ME + mi][ni] : acc[mi][ni];
            }
        __syncthreads();
        const int other = wmn + (wk ? 0 : WGM * WGN);
#pragma unroll
        for (int mi = 0; mi < ME; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) fin[mi][ni] += ex[other * PER + (mi * NI + ni) * 64];
    } else {
#pragma unroll
        for (int mi = 0; mi < ME; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) fin[mi][ni] = acc[mi][ni];
    }

    // ---- bias, residual, store: what the problem asks for is decided once, and each choice is straight-line code.  (Two
    // wavefronts on a SIMD issue an instruction every eight clocks or so: with the choices made per block the
    // ten blocks of a 128x160 tile took 1.6 us.)
    const float alpha = P.alpha;
    const int64_t ldy = P.ldy;
    // (landed long ago; said here once, or the compiler waits piece by piece, for the stores ahead of a piece too)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        asm volatile("" : "+v"(bias[ni]));
#pragma unroll
        for (int mi = 0; mi < (RES ? ME : 0); ++mi) {
            if (RES == RES_F32) asm volatile("" : "+v"(resf[mi][ni]));
            else asm volatile("" : "+v"(resb[mi][ni]));
        }
    }
    constexpr int OUT_BF16 = 0, OUT_F32 = 1, OUT_TRANSPOSED = 2;   // transposed: 16 rows of x are 32 contiguous bytes
    auto store = [&](auto out_kind, auto bounds) {
        constexpr int OK = decltype(out_kind)::v;
        char* const y = static_cast<char*>(P.y) + (OK == OUT_TRANSPOSED ? ((int64_t)ncol * ldy + mrow) * 2 : ((int64_t)mrow * ldy + ncol) * (OK == OUT_F32 ? 4 : 2));
#pragma unroll
        for (int mi = 0; mi < ME; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                f32x4 v = fin[mi][ni];
                v[0] = alpha * v[0] + bf16lo_to_f32(bias[ni][0]);
                v[1] = alpha * v[1] + bf16hi_to_f32(bias[ni][0]);
                v[2] = alpha * v[2] + bf16lo_to_f32(bias[ni][1]);
                v[3] = alpha * v[3] + bf16hi_to_f32(bias[ni][1]);
                if (RES == RES_F32) v += resf[mi][ni];
                if (RES == RES_BF16) {
                    const u32x2 w = resb[mi][ni];
                    v[0] += bf16lo_to_f32(w[0]); v[1] += bf16hi_to_f32(w[0]);
                    v[2] += bf16lo_to_f32(w[1]); v[3] += bf16hi_to_f32(w[1]);
                }
                if (decltype(bounds)::v && !(mrow + mi * 16 < Mp && ncol + ni * 16 < N)) continue;
                if (OK == OUT_F32) {
                    *as_global(reinterpret_cast<f32x4*>(y + mi * ldy * 64 + ni * 64)) = v;
                    continue;
                }
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)v[e];
                if (OK == OUT_BF16) *as_global(reinterpret_cast<bf16x4*>(y + mi * ldy * 32 + ni * 32)) = o;
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e) *as_global(reinterpret_cast<__bf16*>(y + (ni * 16 + e) * ldy * 2 + mi * 32)) = o[e];
            }
    };
    auto by_bounds = [&](auto out_kind) {
        if (m0 + BM <= Mp && n0 + BN <= N) store(out_kind, IntC<0>());
        else store(out_kind, IntC<1>());
    };
    if (RES == RES_NONE && P.bias_on_rows == 2) by_bounds(IntC<OUT_TRANSPOSED>());
    else if (RES != RES_BF16 && P.y_f32) by_bounds(IntC<OUT_F32>());
    else by_bounds(IntC<OUT_BF16>());
}

template <int BM, int BN, int WGM, int WGN, int WGK, int NRB, int DEPTH>
static int launch16(GemmGroup& g, hipStream_t stream) {
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
    if (total == 0 || SD_DRY_RUN("gemm16 %dx%d/%d%s; ", BM, BN, NRB,
                                 dry_detail(", %d problems, %d stages%s", g.n, Tile16<BM, BN, WGM, WGN, WGK, NRB, DEPTH>::STAGES, !g.p[0].res ? "" : g.p[0].res_f32 ? ", fp32 residual" : ", bf16 residual")))
        return SD_OK;
    const dim3 grid((total + 7) & ~7), block(64 * WGM * WGN * WGK);
    if (!g.p[0].res) hipLaunchKernelGGL((gemm16_kernel<BM, BN, WGM, WGN, WGK, NRB, RES_NONE, DEPTH>), grid, block, 0, stream, g);
    else if (g.p[0].res_f32) hipLaunchKernelGGL((gemm16_kernel<BM, BN, WGM, WGN, WGK, NRB, RES_F32, DEPTH>), grid, block, 0, stream, g);
    else hipLaunchKernelGGL((gemm16_kernel<BM, BN, WGM, WGN, WGK, NRB, RES_BF16, DEPTH>), grid, block, 0, stream, g);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}
template <int BM, int BN, int WGM, int WGN, int WGK, int DEPTH = 5>
static int launch16r(GemmGroup& g, int rmax, hipStream_t stream) {
    if (rmax == 0) return launch16<BM, BN, WGM, WGN, WGK, 0, DEPTH>(g, stream);
    if (rmax <= 16 * WGN) return launch16<BM, BN, WGM, WGN, WGK, 1, DEPTH>(g, stream);
    if (rmax <= 32 * WGN) return launch16<BM, BN, WGM, WGN, WGK, 2, DEPTH>(g, stream);
    return launch16<BM, BN, WGM, WGN, WGK, 64 / 16 / WGN, DEPTH>(g, stream);
}

// Which tile, or 0 for the general kernel (any K, rank, layout and alignment; four columns are one access here): the
// largest of the three with which the group is one round of at most one workgroup per CU, and, for the larger two, more
// than half the CUs have one.
//   An adapter costs the tile its A rows in every step (up to rank 32 16 or 32 of them, above 64), the general kernel a
// producer tile, its stores and the wait for them: up to rank 32 the former is cheaper at any K (0.96 to 1.7 times
// as fast over 400 projections of 64 to 16384 rows), of rank 64 while K is short, or where two column tiles are all that repeat it
// (8200x320x1280 + 64 24.3 / 21.1).  (64x80 tiles of rank 64, 77 to 988 rows, K = 1280 to 2560: 0.97 to 1.10 of the general kernel's time,
// of rank 40 0.90 to 1.08, the longer the K loop the worse.)
//   A lone projection that the general kernel fits into one round (128x128 tiles with a deep ring, its producers among them; in
// place of the 64-row tiles its own) is better off there; with an adapter of rank 32 and a short K the 64-row tiles stay ahead.  The q, k, v
// groups always gain: their alternative is three rounds of uneven tiles.
// us, general kernel / here: 512x320x320 + 8 10.4 / 6.1, + 64 9.1 / 7.3; 1000x1280x1280 + 16 13.4 / 9.6, + 64 12.3 / 12.4;
// 3952x640x640 + 16 13.4 / 10.6, + 64 12.7 / 11.3; 8192x640x640 + 64 17.7 / 15.8; 2048x1280x1280 + 64 16.1 / 15.6; 154x1280x2048 + 8
// 14.7 / 10.9, + 64 14.0 / 14.8; 2048x1280x5120 + 32 38.0 / 38.5, + 64 38.8 / 43.8; 4100x640x640 (132 tiles) 11.5 / 14.6, + 16 15.1 / 16.9;
// 6100x640x640 (192) 13.5 / 15.8, + 16 18.4 / 17.7; 8100x640x2560 (256) 36.4 / 32.5, + 16 39.8 / 36.5; the q, k, v and text key / value
// group of 988 tokens of 1280 channels + 16 37.6 / 27.6, of 2 x 256 of 320 + 8 20.4 / 13.9 (values stored transposed).
//   Fewer rows than that: gemm_thin's tiles, the smallest that are one round.  us, here (or the general kernel) / there: 154x1280x2048 9.6 / 5.2, + 8 11.3 / 6.2,
// + 64 14.2 / 8.9; 77x1280x1280 + 32 10.0 / 5.5; 512x320x320 + 8 5.6 / 4.1, x1280 7.5 / 4.4; 32x64: 308x1280x2048 9.8 / 6.9, 1000x320x320 + 8 5.7 / 4.6;
// 64x64, where the K loop is long: 500x1280x5120 21.4 / 19.5, 1000x640x2560 + 16 13.7 / 13.1, 2000x320x1280 7.8 / 7.2 (1000x640x640 + 16 6.9 / 7.0);
// 64x32, for ranks above 32 at any K from 320 on: 736x640x320 + 64 6.9 / 6.5, 602x640x640 + 64 8.3 / 7.6, 405x640x1024 + 64 10.6 / 8.3, 667x640x1280 + 40
// 13.1 / 9.2, 582x640x2048 + 64 13.2 / 12.1, 452x640x5120 + 40 28.5 / 22.1 (120 projections, 0.65 to 0.97).
// They have whole tiles of columns only.  Results with a bias, bf16 and without residual, no layer of a stack asks for: those keep the kernels that they
// had, which is not the faster side (here / there: 154x1280x2048 + 64 14.2 / 8.9, 512x320x320 + 16 5.7 / 4.2, 988x640x2560 + 64 17.7 / 17.7).
constexpr int THIN_32x32 = 4, THIN_32x64 = 5, THIN_64x64 = 6;
static int tile16(const GemmGroup& g) {
    long big = 0, mid = 0, small = 0, general = 0, lead = 0;   // tiles; of the general kernel: 128x128, and its producers'
    long thin[3] = {0, 0, 0};                                  // gemm_thin's: 32x32, 32x64, 64x64 (64x32 above rank 32)
    bool thin_ok = true;
    int rmax = 0, kmax = 0, nmax = 0;
    for (int i = 0; i < g.n; ++i) {
        const GemmProblem& P = g.p[i];
        if (P.geglu_F > 0 || P.bias_on_rows == 1 || P.K0 % 64 || P.K1 > 64 || P.N % 4 || (P.bias_on_rows == 2 ? P.y_f32 || P.res : P.ldy % 4) || (P.res && P.ldr % 4) || P.Mp <= 0 || P.N <= 0 ||
            (uintptr_t)P.bias % 8 || (uintptr_t)P.y % (P.bias_on_rows == 2 ? 2 : P.y_f32 ? 16 : 8) || (uintptr_t)P.res % (P.res_f32 ? 16 : 8) ||
            P.ldp0 * 512 >= (1ll << 31) || P.ldq0 * 512 >= (1ll << 31) || (P.res && g.n > 1))
            return 0;
        big += (long)((P.Mp + 127) / 128) * ((P.N + 159) / 160);
        mid += (long)((P.Mp + 63) / 64) * ((P.N + 159) / 160);
        small += (long)((P.Mp + 63) / 64) * ((P.N + 79) / 80);
        general += (long)((P.Mp + 127) / 128) * ((P.N + 127) / 128);
        lead += (long)((P.Mp + 127) / 128) * ((P.K1 + 63) / 64);
        for (int i = 0; i < 2; ++i) thin[i] += (long)((P.Mp + 31) / 32) * (P.N / (32 << i));
        thin[2] += (long)((P.Mp + 63) / 64) * P.N;             // (columns: how many a tile has is up to the largest rank)
        thin_ok = thin_ok && P.N % 64 == 0 && (!P.bias || P.res || P.y_f32);
        rmax = P.K1 > rmax ? P.K1 : rmax;
        kmax = P.K0 > kmax ? P.K0 : kmax;
        nmax = P.N > nmax ? P.N : nmax;
    }
    thin[2] /= rmax > 32 ? 32 : 64;
    if (thin_ok && kmax >= 320) {
        if (thin[0] <= 256) return THIN_32x32;
        if (thin[1] <= 256 && rmax <= 32) return THIN_32x64;
        if (thin[2] <= 256 && (rmax > 32 || kmax >= 1024)) return THIN_64x64;
    }
    const int tile = big <= 256 && big > 128 ? 3 : mid <= 256 && mid > 128 ? 2 : small <= 256 ? 1 : 0;
    if (rmax > 32 && kmax > 640 && !(nmax <= 320 && tile > 1)) return 0;
    if (g.n == 1 && tile == 3 && gemm_one_round(general, lead)) return 0;
    if (g.n == 1 && tile == 2 && general <= 128 && general + lead <= 140 && !(rmax > 0 && rmax <= 32 && kmax <= 640)) return 0;
    return tile;
}
bool gemm16_takes(const GemmGroup& g) { return tile16(g) > 0; }
int launch_gemm16(GemmGroup& g, hipStream_t stream) {
    int rmax = 0, kmax = 0;
    for (int i = 0; i < g.n; ++i) {
        rmax = g.p[i].K1 > rmax ? g.p[i].K1 : rmax;
        kmax = g.p[i].K0 > kmax ? g.p[i].K0 : kmax;
    }
    const int tile = tile16(g);
    switch (tile) {
    case THIN_32x32:
    case THIN_32x64:
    case THIN_64x64: return launch_gemm_thin(g, tile - THIN_32x32, stream);
    case 3: return launch16r<128, 160, 4, 2, 1>(g, rmax, stream);
    case 2: return launch16r<64, 160, 2, 2, 2>(g, rmax, stream);
    // One workgroup of four wavefronts per CU: the two stages that three leave in flight (37 KB) come in at 54 GB/s, the latency of
    // the last-level cache.  Four take 15 % off a long K loop and more first loads in front of a short one.  988 rows of 1280 columns + 8, us,
    // three / four stages, weights from the last-level cache: K = 5120 29.4 / 25.6, 2048 13.4 / 12.7, 1280 10.2 / 9.8; in L2 from a call
    // before: 26.8 / 22.6, 11.1 / 11.4, 8.8 / 9.1; K = 640 without adapter 7.2 / 7.3.  (512 rows of 320x320 + 8 5.5 / 5.7, 1000 of 640x640 + 64 8.6 / 9.2; five
    // stages 0.1 to 0.3 more than four.  Four wavefronts more that split K in four took as much off and cost 1 us in front.)
    default:
        if (kmax <= 640) return launch16r<64, 80, 2, 1, 2, 3>(g, rmax, stream);
        if (rmax == 0) return launch16<64, 80, 2, 1, 2, 0, 4>(g, stream);
        if (rmax <= 16) return launch16<64, 80, 2, 1, 2, 1, 4>(g, stream);
        return launch16<64, 80, 2, 1, 2, 2, 4>(g, stream);     // (above rank 32 this tile is for K <= 640)
    }
}

}  // namespace sd
