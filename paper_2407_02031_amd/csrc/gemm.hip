// Grouped bf16 MFMA GEMM for gfx950 with the rank-r LoRA update fused into the main loop.
//
// Every projection of the transformer block is y = x W^T (+ bias) with an optional LoRA
// term scale * (x A^T) B^T (Section 2, "Low-Rank Adaptation").  The down-projection
// t = scale * x A^T is a small GEMM of its own; the up-projection then rides in the base
// GEMM's K loop: [x | t] [W | B]^T, i.e. a second K segment of length r.  Both run in one
// launch: the down-projection's tiles come first in the grid and raise a flag per row block,
// and a base-GEMM tile looks at its flag only when it reaches the second K segment.
// Epilogues: bias, exact-erf GEGLU (Section 4.3's fused GEGLU), residual add, bf16 or fp32
// store.
//
// Tiling: BM x BN output tile per workgroup, BK = 64, WGM x WGN wavefronts, each owning
// (BM/WGM) x (BN/WGN) as 16x16x32 bf16 MFMA tiles with fp32 accumulators (32x32x16 ones cost more
// energy, and the chip lowers its clock under them: 8192x4096x4096 223 -> 211 us, 16384x1280x5120 + 64 249 -> 240, 8 x 4096 rows of
// 640 channels with four adapters 43.4 -> 42.6, 5000x640x2560 + 64 28.4 -> 26.8; same bits.  Some of the launches with one tile per CU are slower, and why is not known:
// 3000x1280x5120 + 64 55.5 -> 57.7, 6000x640x1280 + 64 21.0 -> 21.6, 4120x640x320 + 64 10.7 -> 10.9).
// Pipeline: operand tiles go global -> LDS directly (wave-wide 1 KB loads of 16-byte
// chunks, XOR-swizzled so the 16 rows one MFMA operand read touches fall in distinct
// banks) into a ring of STAGES tiles, STAGES-1 of them in flight ahead of the one being
// multiplied; operand blocks are read from LDS a few MFMAs ahead of their use,
// across the edge of two tiles too, and a tile's loads are dealt between the MFMAs of a
// step.  What bounds it: the L2 -> LDS operand stream, 100-125 GB/s per CU with all of them at it
// (a stream alone: 145 with few CUs), then the MFMAs, whose rate under load is 1.6 PFLOP/s; the
// two overlap only as far as no wavefront waits to issue a load.  8192x4096x4096, 128x128 tiles,
// eight wavefronts, three loads a burst after each barrier 271 us, dealt 248; 2048x1280x5120 + 64
// at one 128x128 tile per CU 51 and 41.  The epilogue stages 32-row x 64-column pieces of a wave's
// accumulators through LDS so that global stores (and residual loads) are 16-byte rows.
#include "gemm_dma.hpp"

namespace sd {

constexpr int EPI_STRIDE = 68;   // floats per staged row: 16 rows apart by 4 banks, 16 bytes of each

// Tiles that gave up waiting for a producer's flag (never, unless the dependency protocol is
// broken): the wait is bounded so that every wavefront exits whatever happens.
__device__ unsigned long long g_gemm_dep_timeouts = 0;
constexpr int DEP_SPIN_LIMIT = 1 << 19;
struct DeviceMem {
    __device__ __forceinline__ static uint64_t load64(const uint64_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ static void store64(uint64_t* p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ static void store32(int32_t* p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ static int32_t add32(int32_t* p, int32_t v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};
// Tiles of signalling problems (down-projections, N = rank) run a body of their own inside the
// same kernel: BN = 64 instead of the launch's BN, which frees LDS for a deeper ring.  Other
// tiles of the launch wait for these, and what a down-projection tile spends is latency per
// k-step, so tiles in flight are what shortens it.
constexpr int DOWN_BN = 64;
template <int BM, int BN, int BK, int STAGES>
constexpr int down_stages() {
    if (BN <= DOWN_BN) return STAGES;
    const int fit = STAGES * (BM + BN) / (BM + DOWN_BN);   // stages of the narrower tile in the same bytes
    return fit > 5 ? 5 : (fit < 3 ? 3 : fit);
}
template <int BM, int BN, int BK, int WGM, int WGN, int STAGES>
constexpr int gemm_lds_chunks() {
    constexpr int ring = STAGES * (BM + BN) * (BK / 8);
    constexpr int dring = down_stages<BM, BN, BK, STAGES>() * (BM + (BN < DOWN_BN ? BN : DOWN_BN)) * (BK / 8);
    constexpr int epi = WGM * WGN * 32 * EPI_STRIDE / 4;
    constexpr int m = ring > dring ? ring : dring;
    return m > epi ? m : epi;
}

// GUARD: K segments that are not multiples of 64 (tail chunks read zeros).
// Two workgroups per CU whenever the ring leaves room for it (LDS <= 80 KB): the register
// budget is then 256 per lane (accumulators in AGPRs, the rest in VGPRs).
template <int BM, int BN, int BK, int WGM, int WGN, int STAGES>
constexpr int gemm_min_waves() {
    return gemm_lds_chunks<BM, BN, BK, WGM, WGN, STAGES>() * 16 <= 80 * 1024 ? 2 : 1;
}

template <int BM, int BN, int BK, int WGM, int WGN, int STAGES, bool GEGLU, bool GUARD, bool RES32>
__device__ __forceinline__ void gemm_tile(const GemmProblem& P, const int tile, u32x4* const lds) {
    constexpr int NW = WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int MI = WM / 16, NI = WN / 16;  // 16x16 blocks of a wavefront
    constexpr int CPR = BK / 8;                // 16-byte chunks per LDS row
    constexpr int RPB = 64 / CPR;              // tile rows per 1 KB block (one wave-wide load)
    constexpr int SLOTS = 2 * NI;              // a tile is two 32 deep k-steps of NI blocks of Q; a slot multiplies one of them by the MI blocks of P
    constexpr int RING = NI < 4 ? NI : 4;      // blocks of Q in registers
    constexpr int NBLK = (BM + BN) / RPB;      // 1 KB blocks per stage
    constexpr int LPT = NBLK / NW;             // direct-to-LDS loads per wave (= per lane) per tile
    constexpr int STAGE = (BM + BN) * CPR;     // 16-byte chunks per stage
    static_assert(BK == 64 && SLOTS % RING == 0, "BK");
    static_assert(NBLK % NW == 0, "tile/waves mismatch");
    static_assert(!GEGLU || (NI % 2 == 0), "GEGLU needs value/gate column-block pairs per wave");
    static_assert(STAGES >= 2 && STAGES <= 5, "ring depth");

    // ---- which tile of the problem ----
    const int local = tile - P.tile_begin;
    const int band_tiles = 8 * P.tiles_n;
    const int band = local / band_tiles, rem = local - band * band_tiles;
    const int band_rows = min(8, P.tiles_m - band * 8);
    const int tn = rem / band_rows, tm = band * 8 + rem % band_rows;
    constexpr int BN_OUT = GEGLU ? BN / 2 : BN;
    const int m0 = tm * BM, n0 = tn * BN_OUT;
    const int Mp = P.Mp, N = P.N, K0 = P.K0, K1 = P.K1;
    const int nk0 = (K0 + BK - 1) / BK, nk1 = (K1 + BK - 1) / BK, nkt = nk0 + nk1;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int wm = (wave / WGN) * WM, wn = (wave % WGN) * WN;

    // ---- dependency on a producer problem of this launch.  The flags are read once now (the
    // answer arrives with the first operand tile); tiles that start after the producer has
    // finished, the usual case, never look again.  Device-scope loads: the producer's tile may
    // have run on another XCD.
    const int32_t* const wflag = K1 ? P.wait : nullptr;
    const int32_t* fptr = nullptr;
    // with a nonce: the record of this row block, and the word of it that this lane looks at
    uint64_t* const rec = wflag && P.nonce ? reinterpret_cast<uint64_t*>(const_cast<int32_t*>(wflag)) + tm * (DEP_RECORD / 8) : nullptr;
    const uint64_t* const rword = rec + dep_record_word(lane, P.wait_need);
    bool f_early = true;
    if (rec) {
        f_early = dep_record_ready(lane, P.wait_need, DeviceMem::load64(rword), P.nonce);
    } else if (wflag) {
        const int lo = P.wait_cols ? n0 : m0;
        const int hi = P.wait_cols ? min(n0 + BN_OUT, N) : min(m0 + BM, Mp);
        const int f0 = lo / BM, f1 = (hi - 1) / BM;
        fptr = wflag + f0 + min(lane, f1 - f0);
        f_early = __hip_atomic_load(fptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= P.wait_need;
    }

    // Q-operand (weight) row of tile row j.  GEGLU: 16-row blocks alternate value / gate
    // rows of the same 16 output columns, so one lane ends up holding both halves.
    auto qrow = [&](int j) -> int {
        if (GEGLU) {
            int blk = j >> 4;
            int col = n0 + (blk >> 1) * 16 + (j & 15);
            col = col < N ? col : N - 1;
            return col + ((blk & 1) ? P.geglu_F : 0);
        } else {
            int col = n0 + j;
            return col < N ? col : N - 1;
        }
    };

    // ---- loader.  Load j of wave w fills 1 KB block (j*NW + w) of a stage: RPB tile rows
    // (P rows first, then Q rows) of CPR chunks; lane l lands at chunk position l % CPR of row
    // l / CPR, so it must fetch the logical chunk that the XOR swizzle places there.  The
    // first JP loads of a lane are P rows, the rest Q rows; a lane's source is a wave-uniform
    // base (operand start + k offset of the step, scalar arithmetic) plus a constant 32-bit
    // byte offset (row, chunk).
    constexpr int JP = (BM / RPB) / NW;
    static_assert((BM / RPB) % NW == 0, "P/Q split must fall on a load index");
    uint32_t off0[LPT];          // byte offset of this lane's chunk from the operand start, K segment 0
    uint32_t off1[LPT];          // ... K segment 1 (LoRA); equals off0 when there is none
    int kcol[GUARD ? LPT : 1];   // first k of that chunk within a tile (only partial tiles need it)
    const uint16_t* const pb0 = P.p0 + (int64_t)m0 * P.ldp0;
    const uint16_t* const pb1 = K1 ? P.p1 + (int64_t)m0 * P.ldp1 : pb0;
    const uint16_t* const qb0 = P.q0 + (int64_t)n0 * P.ldq0;
    const uint16_t* const qb1 = K1 ? P.q1 + (int64_t)n0 * P.ldq1 : qb0;
    {
        const int64_t ldp0 = P.ldp0, ldq0 = P.ldq0;
        const int64_t ldp1 = K1 ? P.ldp1 : P.ldp0, ldq1 = K1 ? P.ldq1 : P.ldq0;
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const int row = (j * NW + wave) * RPB + lane / CPR;    // row within the stage
            const int c = swz<CPR>(row, lane % CPR);               // logical chunk fetched by this lane
            if (GUARD) kcol[j] = c * 8;
            if (j < JP) {
                int r = m0 + row;
                r = (r < Mp ? r : Mp - 1) - m0;
                off0[j] = (uint32_t)((r * ldp0 + c * 8) * 2);
                off1[j] = (uint32_t)((r * ldp1 + c * 8) * 2);
            } else {
                const int qr = qrow(row - BM) - n0;
                off0[j] = (uint32_t)((qr * ldq0 + c * 8) * 2);
                off1[j] = (uint32_t)((qr * ldq1 + c * 8) * 2);
            }
        }
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    const uint32_t wave_base = lds_base + (uint32_t)wave * 1024;
    // issue the loads of k-step t into ring stage `stg`.  A partial last tile of a segment
    // (GUARD only) takes per-lane 64-bit addresses so that chunks past the segment's end can
    // point at the zero page.
    bool dep_ready = wflag == nullptr;
    bool timed_out = false;      // this wavefront gave up waiting: its output is poisoned below
    auto issue_tile = [&](int t, int stg) {
        const bool s1 = t >= nk0;
        const int kb = (s1 ? t - nk0 : t) * BK;
        const int Kseg = s1 ? K1 : K0;
        const uint32_t sbase = wave_base + (uint32_t)stg * (STAGE * 16);
        const uint16_t* pb = (s1 ? pb1 : pb0) + kb;
        const uint16_t* qb = (s1 ? qb1 : qb0) + kb;
        const bool dev = s1 && wflag;   // segment 1 was written during this launch
        if (dev && !dep_ready) {
            // the producer's tiles were dispatched before this one and wait for nothing, so
            // this ends; the bound is there so that it ends even if that reasoning is wrong
            for (int spins = 0;; ++spins) {
                bool seen, given_up = false;
                if (rec) {
                    const uint64_t v = DeviceMem::load64(rword);
                    seen = dep_record_ready(lane, P.wait_need, v, P.nonce);
                    given_up = dep_record_given_up(lane, P.wait_need, v, P.nonce);
                } else {
                    seen = __hip_atomic_load(fptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= P.wait_need;
                }
                if (__all(seen)) break;
                if (spins >= DEP_SPIN_LIMIT || __any(given_up)) {
                    if (tid == 0) atomicAdd(&g_gemm_dep_timeouts, 1ull);
                    if (rec && lane == 0) DepRecord<DeviceMem>::give_up(rec, P.nonce);
                    timed_out = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(8);
            }
            dep_ready = true;
        }
        if (GUARD && kb + BK > Kseg) {
#pragma unroll
            for (int j = 0; j < LPT; ++j) {
                const char* src = reinterpret_cast<const char*>(j < JP ? pb : qb) + (s1 ? off1[j] : off0[j]);
                src = (kb + kcol[GUARD ? j : 0] < Kseg) ? src : reinterpret_cast<const char*>(g_gemm_zeros);
                if (dev) dma16<true>(src, sbase + (uint32_t)j * (NW * 1024));
                else dma16<false>(src, sbase + (uint32_t)j * (NW * 1024));
            }
        } else if (dev) {
#pragma unroll
            for (int j = 0; j < LPT; ++j)
                dma16_so<true>(j < JP ? pb : qb, off1[j], sbase + (uint32_t)j * (NW * 1024));
        } else {
#pragma unroll
            for (int j = 0; j < LPT; ++j)
                dma16_so<false>(j < JP ? pb : qb, s1 ? off1[j] : off0[j], sbase + (uint32_t)j * (NW * 1024));
        }
    };

    f32x4 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

    // operands in registers: the P blocks of both k-steps, and a ring of Q blocks.  Slot s multiplies Q block s % NI in k-step
    // s / NI out of bfr[s % RING], which is then refilled for slot s + RING, over the edge between two tiles too.
    // The MFMA takes the Q rows first: a lane holds four consecutive columns of one row of the result.
    bf16x8 af[2][MI], bfr[RING];
    const int lrow = l16 * CPR, lsw = (l16 >> 1) & 7;       // (rows 16 apart share the swizzle)
    auto frag = [&](int st, int ks) { return lds + (st * STAGE + lrow + ((ks * 4 + quad) ^ lsw)); };
    auto fetch_p = [&](int st, int ks) {
        const u32x4* const la = frag(st, ks) + wm * CPR;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) af[ks][mi] = __builtin_bit_cast(bf16x8, la[mi * 16 * CPR]);
    };
    auto fetch_q = [&](int st, int s) { bfr[s % RING] = __builtin_bit_cast(bf16x8, (frag(st, s / NI) + (BM + wn) * CPR)[(s % NI) * 16 * CPR]); };
    auto multiply = [&](int s) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            acc[mi][s % NI] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[s % RING], af[s / NI][mi], acc[mi][s % NI], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // A step: the last RING slots of a tile, whose operands are in registers, while the first of the next (in stage sn) are read
    // (`edge`); then the others of that one (`head`).  The loads of another tile are dealt over it, a few behind each
    // slot's MFMAs (`load(j)` issues one): a wavefront issues in order, and a burst of loads would hold up its
    // MFMAs until the address unit has taken the last one, at 16 clocks apiece for the whole CU.
    auto deal = [&](auto load, int i) {
#pragma unroll
        for (int j = i * LPT / SLOTS; j < (i + 1) * LPT / SLOTS; ++j) load(j);
    };
    auto edge = [&](int sn, auto load) {
        fetch_p(sn, 0);
#pragma unroll
        for (int i = 0; i < RING; ++i) {
            multiply(SLOTS - RING + i);
            deal(load, i);
            fetch_q(sn, i);
        }
    };
    auto head = [&](int st, auto load) {
#pragma unroll
        for (int s = 0; s < SLOTS - RING; ++s) {
            if (s == 0) fetch_p(st, 1);
            multiply(s);
            deal(load, RING + s);
            fetch_q(st, s + RING);
        }
    };
    auto no_load = [](int) {};

    // ---- prologue: the first STAGES tiles in flight, the first fragments of tile 0 read
#pragma unroll
    for (int d = 0; d < STAGES; ++d)
        if (d < nkt) issue_tile(d, d);
    if (!dep_ready) dep_ready = __all(f_early);
    auto wait_tiles = [&](int newer) {   // `newer` tiles (at most STAGES - 1) may stay in flight
        if (STAGES >= 5 && newer >= 4) wait_vmcnt<4 * LPT>();
        else if (STAGES >= 4 && newer >= 3) wait_vmcnt<3 * LPT>();
        else if (STAGES >= 3 && newer >= 2) wait_vmcnt<2 * LPT>();
        else if (newer >= 1) wait_vmcnt<LPT>();
        else wait_vmcnt<0>();
    };
    wait_tiles(nkt - 1 < STAGES - 1 ? nkt - 1 : STAGES - 1);
    __syncthreads();
    fetch_p(0, 0);
#pragma unroll
    for (int s = 0; s < RING; ++s) fetch_q(0, s);
    head(0, no_load);

    // ---- main loop.  A step starts at the edge between tile t and tile t+1, before the MFMAs of
    // tile t's last slots: their operands are in registers, so once this wave's loads of tile t+1
    // have landed (newer ones may stay in flight) one barrier says both that tile t+1 is whole and
    // that the stage of tile t is free.  That stage is refilled with tile t+STAGES, its loads dealt
    // over the step.
    int st = 0;                         // stage of tile t
    int t = 0;
    const int nfull = GUARD ? K0 / BK : nk0;   // whole tiles of K segment 0
#pragma unroll 1
    for (; t + STAGES < nfull; ++t) {
        wait_vmcnt<(STAGES - 2) * LPT>();
        __syncthreads();
        const int sn = st + 1 == STAGES ? 0 : st + 1;
        const uint16_t* const pb = pb0 + (t + STAGES) * BK;
        const uint16_t* const qb = qb0 + (t + STAGES) * BK;
        const uint32_t sbase = wave_base + (uint32_t)st * (STAGE * 16);
        auto load = [&](int j) { dma16_so<false>(j < JP ? pb : qb, off0[j], sbase + (uint32_t)j * (NW * 1024)); };
        edge(sn, load);
        head(sn, load);
        st = sn;
    }
    // the same for the tiles around and behind the end of segment 0, and for the last ones, which
    // have nothing left to load and shrinking wait counts
#pragma unroll 1
    for (; t + 1 < nkt; ++t) {
        wait_tiles(nkt - 2 - t < STAGES - 2 ? nkt - 2 - t : STAGES - 2);
        __syncthreads();
        const int sn = st + 1 == STAGES ? 0 : st + 1;
        if (t + STAGES < nkt) issue_tile(t + STAGES, st);
        edge(sn, no_load);
        head(sn, no_load);
        st = sn;
    }

    // ---- epilogue geometry.  A lane holds columns 4*quad .. +4 of each of its 16-column blocks, in row l16 of each 16-row block.
    // Each wave stages a 32-row x CCOLS-column piece at a time in its own LDS region (fp32, padded rows) and writes it out as
    // whole row pieces: lane handles 4 consecutive columns (lcol) of row lr, lr + RPP, ... of the piece.  (Stored from where they are, 32 or 64 bytes
    // of a row at a time: 8192x1920x640 + 64 39 -> 44 us, 2048x1280x1280 + 64 with an fp32 residual 20.1 -> 21.9.)
    constexpr int NOUT = GEGLU ? NI / 2 : NI;   // 16-column output blocks per wave
    constexpr int CB = (NOUT % 4 == 0) ? 4 : 2; // ... staged per pass (<= 64 columns)
    constexpr int CCOLS = CB * 16;              // staged columns
    constexpr int LPR = CCOLS / 4;              // lanes per staged row (4 columns each)
    constexpr int RPP = 64 / LPR;               // rows per pass
    constexpr int NPASS = 32 / RPP;
    static_assert(NOUT % CB == 0 && MI % 2 == 0, "pieces");
    const int wn_out = GEGLU ? (wn >> 1) : wn;
    const bool y_f32 = P.y_f32 != 0;
    const int lr = lane / LPR, lcol = (lane % LPR) * 4;
    const bool ld_ok = ((P.ldy & 3) == 0) && (!P.res || (P.ldr & 3) == 0);
    // a tile that lies inside the output with 16-byte-aligned rows takes straight-line code: all
    // staged pieces read, then all residual pieces, then all stores (no per-lane bounds)
    const bool full = ld_ok && m0 + BM <= Mp && n0 + BN_OUT <= N;
    const int qcol = n0 + wn_out + quad * 4;

    // fp32 residual: fetch this lane's pieces of the whole wave tile now, so that the loads
    // fly during the last tile's MFMAs and the epilogue never waits piece by piece
    f32x4 rpre[RES32 ? MI / 2 : 1][RES32 ? NOUT / CB : 1][RES32 ? NPASS : 1];
    const bool res_pre = RES32 && P.res && P.res_f32 && ld_ok;
    if (RES32 && res_pre) {
        const float* rp = static_cast<const float*>(P.res);
#pragma unroll
        for (int mi = 0; mi < MI / 2; ++mi)
#pragma unroll
            for (int cc = 0; cc < NOUT / CB; ++cc) {
                const int q4 = n0 + wn_out + cc * CCOLS + lcol;
#pragma unroll
                for (int pass = 0; pass < NPASS; ++pass) {
                    const int p = m0 + wm + mi * 32 + pass * RPP + lr;
                    f32x4 r = {0.f, 0.f, 0.f, 0.f};
                    if (p < Mp && q4 + 4 <= N) r = *reinterpret_cast<const f32x4*>(rp + (int64_t)p * P.ldr + q4);
                    rpre[RES32 ? mi : 0][RES32 ? cc : 0][RES32 ? pass : 0] = r;
                }
            }
    }
    // per-column bias of this lane's output columns: fetched now as well (raw bits, widened after
    // the last MFMAs; a column past N reads the last valid one and is never stored)
    const uint16_t* bias = P.bias;
    u32x2 bv_raw[NOUT], bg_raw[GEGLU ? NOUT : 1];
#pragma unroll
    for (int nj = 0; nj < NOUT; ++nj) {
        bv_raw[nj] = u32x2{0u, 0u};
        if (GEGLU) bg_raw[GEGLU ? nj : 0] = u32x2{0u, 0u};
    }
    if (bias && !P.bias_on_rows) {
        // (a record's bias need not be aligned; whole pieces of four where it is)
        const bool pieces = n0 + BN_OUT <= N && ((reinterpret_cast<uintptr_t>(bias) & 7) == 0) && (!GEGLU || (P.geglu_F & 3) == 0);
        auto four = [&](const uint16_t* b, int q4) {
            if (pieces) return *as_global(reinterpret_cast<const u32x2*>(b + q4));
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = *as_global(b + min(q4 + e, N - 1));
            return u32x2{w[0] | (w[1] << 16), w[2] | (w[3] << 16)};
        };
#pragma unroll
        for (int nj = 0; nj < NOUT; ++nj) {
            bv_raw[nj] = four(bias, qcol + nj * 16);
            if (GEGLU) bg_raw[GEGLU ? nj : 0] = four(bias + P.geglu_F, qcol + nj * 16);
        }
    }
#pragma unroll
    for (int s = SLOTS - RING; s < SLOTS; ++s) multiply(s);
    __syncthreads();   // ring reads done before the epilogue reuses LDS
    // a record's last reader takes the nonce out again.  (Every wavefront of the tile has seen the words by
    // now, or has given up; the count was zeroed before the first of them was written.)
    int readers_before = -1;
    if (rec && tid == 0) readers_before = DepRecord<DeviceMem>::leave(rec);

    // ---- epilogue
    float* stage = reinterpret_cast<float*>(lds) + wave * 32 * EPI_STRIDE;
    // a wavefront that read its second K segment without the producer's flag stores NaN: what it
    // computed from a stale or half-written down-projection must not look like a result
    const float alpha = timed_out ? __builtin_nanf("") : P.alpha;
    int32_t* const sig = P.signal;
    // (opaque to the optimiser, which would otherwise widen right after the loads and wait for them there)
#pragma unroll
    for (int nj = 0; nj < NOUT; ++nj) {
        asm volatile("" : "+v"(bv_raw[nj]));
        if (GEGLU) asm volatile("" : "+v"(bg_raw[GEGLU ? nj : 0]));
    }
    auto widen = [](const u32x2& w, int e) { return e & 1 ? bf16hi_to_f32(w[e >> 1]) : bf16lo_to_f32(w[e >> 1]); };
    // block (mi, nj) as it is staged
    auto value = [&](int mi, int nj) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (GEGLU) v[e] = (alpha * acc[mi][GEGLU ? 2 * nj : 0][e] + widen(bv_raw[nj], e)) * gelu_erf(alpha * acc[mi][GEGLU ? 2 * nj + 1 : 0][e] + widen(bg_raw[GEGLU ? nj : 0], e));
            else v[e] = alpha * acc[mi][nj][e] + widen(bv_raw[nj], e);
        }
        return v;
    };
#pragma unroll
    for (int mi = 0; mi < MI / 2; ++mi) {
#pragma unroll
        for (int cc = 0; cc < NOUT / CB; ++cc) {
            // 1) registers -> staging (value after alpha, bias, GEGLU)
#pragma unroll
            for (int m2 = 0; m2 < 2; ++m2)
#pragma unroll
                for (int cj = 0; cj < CB; ++cj)
                    *reinterpret_cast<f32x4*>(stage + (m2 * 16 + l16) * EPI_STRIDE + cj * 16 + quad * 4) = value(mi * 2 + m2, cc * CB + cj);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // 2) staging -> global: lane handles 4 consecutive columns of one row per pass
            const int q4 = n0 + wn_out + cc * CCOLS + lcol;
            if (full) {
                f32x4 val[NPASS];
#pragma unroll
                for (int pass = 0; pass < NPASS; ++pass)
                    val[pass] = *reinterpret_cast<const f32x4*>(stage + (pass * RPP + lr) * EPI_STRIDE + lcol);
                const int p0 = m0 + wm + mi * 32 + lr;          // row of pass 0; pass k is RPP * k rows further
                if (bias && P.bias_on_rows) {
                    float br[NPASS];
#pragma unroll
                    for (int pass = 0; pass < NPASS; ++pass) br[pass] = bf16_to_f32(bias[p0 + pass * RPP]);
#pragma unroll
                    for (int pass = 0; pass < NPASS; ++pass) val[pass] += br[pass];
                }
                if (P.res) {
                    if (RES32 && res_pre) {
#pragma unroll
                        for (int pass = 0; pass < NPASS; ++pass) val[pass] += rpre[RES32 ? mi : 0][RES32 ? cc : 0][RES32 ? pass : 0];
                    } else if (P.res_f32) {
                        const float* rf = static_cast<const float*>(P.res) + (int64_t)p0 * P.ldr + q4;
                        f32x4 r[NPASS];
#pragma unroll
                        for (int pass = 0; pass < NPASS; ++pass) r[pass] = *reinterpret_cast<const f32x4*>(rf + (int64_t)(pass * RPP) * P.ldr);
#pragma unroll
                        for (int pass = 0; pass < NPASS; ++pass) val[pass] += r[pass];
                    } else {
                        const uint16_t* rb = static_cast<const uint16_t*>(P.res) + (int64_t)p0 * P.ldr + q4;
                        u32x2 r[NPASS];
#pragma unroll
                        for (int pass = 0; pass < NPASS; ++pass) r[pass] = *reinterpret_cast<const u32x2*>(rb + (int64_t)(pass * RPP) * P.ldr);
#pragma unroll
                        for (int pass = 0; pass < NPASS; ++pass) {
                            val[pass][0] += bf16lo_to_f32(r[pass][0]); val[pass][1] += bf16hi_to_f32(r[pass][0]);
                            val[pass][2] += bf16lo_to_f32(r[pass][1]); val[pass][3] += bf16hi_to_f32(r[pass][1]);
                        }
                    }
                }
                if (y_f32) {
                    float* yp = static_cast<float*>(P.y) + (int64_t)p0 * P.ldy + q4;
#pragma unroll
                    for (int pass = 0; pass < NPASS; ++pass) *reinterpret_cast<f32x4*>(yp + (int64_t)(pass * RPP) * P.ldy) = val[pass];
                } else {
                    uint16_t* yp = static_cast<uint16_t*>(P.y) + (int64_t)p0 * P.ldy + q4;
#pragma unroll
                    for (int pass = 0; pass < NPASS; ++pass) {
                        bf16x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = (__bf16)val[pass][e];
                        uint16_t* const yq = yp + (int64_t)(pass * RPP) * P.ldy;
                        if (sig)   // device-scope store: read by tiles of this launch on other XCDs
                            __hip_atomic_store(reinterpret_cast<uint64_t*>(yq), __builtin_bit_cast(uint64_t, o), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                        else
                            *reinterpret_cast<bf16x4*>(yq) = o;
                    }
                }
            } else {
                const bool vec_ok = ld_ok && (q4 + 4 <= N);   // 16-byte path: whole piece inside N, aligned rows
#pragma unroll
                for (int pass = 0; pass < NPASS; ++pass) {
                    const int rr = pass * RPP + lr;
                    const int p = m0 + wm + mi * 32 + rr;
                    if (p < Mp && q4 < N) {
                        f32x4 val = *reinterpret_cast<const f32x4*>(stage + rr * EPI_STRIDE + lcol);
                        if (bias && P.bias_on_rows) val += bf16_to_f32(bias[p]);
                        const int64_t oi = (int64_t)p * P.ldy + q4;
                        const int64_t ri = (int64_t)p * P.ldr + q4;
                        if (y_f32) {
                            float* yp = static_cast<float*>(P.y) + oi;
                            const float* rp = static_cast<const float*>(P.res);
                            if (vec_ok) {
                                if (RES32 && res_pre) val += rpre[RES32 ? mi : 0][RES32 ? cc : 0][RES32 ? pass : 0];
                                else if (rp) val += *reinterpret_cast<const f32x4*>(rp + ri);
                                *reinterpret_cast<f32x4*>(yp) = val;
                            } else {
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    if (q4 + e < N) yp[e] = val[e] + (rp ? rp[ri + e] : 0.f);
                            }
                        } else {
                            uint16_t* yp = static_cast<uint16_t*>(P.y) + oi;
                            const uint16_t* rp = static_cast<const uint16_t*>(P.res);
                            if (P.res_f32 && rp) {      // fp32 residual stream into a bf16 output
                                const float* rf = static_cast<const float*>(P.res);
                                if (RES32 && res_pre) val += rpre[RES32 ? mi : 0][RES32 ? cc : 0][RES32 ? pass : 0];
                                else if (vec_ok) val += *reinterpret_cast<const f32x4*>(rf + ri);
                                else
#pragma unroll
                                    for (int e = 0; e < 4; ++e)
                                        if (q4 + e < N) val[e] += rf[ri + e];
                                rp = nullptr;
                            }
                            if (vec_ok) {
                                if (rp) {
                                    const u32x2 rv = *reinterpret_cast<const u32x2*>(rp + ri);
                                    val[0] += bf16lo_to_f32(rv[0]); val[1] += bf16hi_to_f32(rv[0]);
                                    val[2] += bf16lo_to_f32(rv[1]); val[3] += bf16hi_to_f32(rv[1]);
                                }
                                bf16x4 o;
#pragma unroll
                                for (int e = 0; e < 4; ++e) o[e] = (__bf16)val[e];
                                if (sig)   // device-scope store: read by tiles of this launch on other XCDs
                                    __hip_atomic_store(reinterpret_cast<uint64_t*>(yp), __builtin_bit_cast(uint64_t, o), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
                                else
                                    *reinterpret_cast<bf16x4*>(yp) = o;
                            } else {
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    if (q4 + e < N) {
                                        const float f = val[e] + (rp ? bf16_to_f32(rp[ri + e]) : 0.f);
                                        yp[e] = __builtin_bit_cast(uint16_t, (__bf16)f);
                                    }
                            }
                        }
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (rec && tid == 0 && readers_before == P.readers - 1) DepRecord<DeviceMem>::clear(rec);
    // ---- tell the tiles that wait for this one: every wave's stores have completed at device
    // scope (vmcnt counts a device-scope store until it is visible there), then one flag add, or
    // the nonce in this column tile's word
    if (sig && P.nonce) {
        uint64_t* const w = reinterpret_cast<uint64_t*>(sig) + tm * (DEP_RECORD / 8);
        if (tid == 0) DepRecord<DeviceMem>::open(w, tn);
        wait_vmcnt<0>();
        __syncthreads();
        if (tid == 0) DepRecord<DeviceMem>::publish(w, tn, P.nonce);
    } else if (sig) {
        wait_vmcnt<0>();
        __syncthreads();
        if (tid == 0) __hip_atomic_fetch_add(sig + tm, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int BM, int BN, int BK, int WGM, int WGN, int STAGES, bool GEGLU, bool GUARD, bool RES32>
__global__ __launch_bounds__(64 * WGM * WGN, (gemm_min_waves<BM, BN, BK, WGM, WGN, STAGES>())) void gemm_kernel(const GemmGroup g) {
    constexpr int NW = WGM * WGN;
    __shared__ u32x4 lds[gemm_lds_chunks<BM, BN, BK, WGM, WGN, STAGES>()];
    GemmProblem P;
    int tile, zero_n;
    int32_t* zero_ptr;
    const bool any = gemm_pick_tile(g, tile, P, zero_n, zero_ptr);
    // flags of the next dependent launch, a few words per workgroup: nothing reads them before this kernel ends
    for (int i = blockIdx.x * (64 * NW) + threadIdx.x; i < zero_n; i += (int)gridDim.x * (64 * NW)) zero_ptr[i] = 0;
    if (!any) return;
    if constexpr (BN > DOWN_BN) {
        if (P.signal) {
            gemm_tile<BM, DOWN_BN, BK, WGM * WGN / 2, 2, down_stages<BM, BN, BK, STAGES>(), false, GUARD, false>(P, tile, lds);
            return;
        }
    }
    gemm_tile<BM, BN, BK, WGM, WGN, STAGES, GEGLU, GUARD, RES32>(P, tile, lds);
}

template <int BM, int BN, int BK, int WGM, int WGN, int STAGES, bool GEGLU, bool RES32>
static int launch_cfg(GemmGroup& g, bool guard, hipStream_t stream) {
    constexpr int BN_OUT = GEGLU ? BN / 2 : BN;
    int total = 0;
    g.n_lead = 0;
    for (int i = 0; i < g.n; ++i) {
        GemmProblem& P = g.p[i];
        P.tiles_m = (P.Mp + BM - 1) / BM;
        P.tiles_n = P.signal ? (P.N + (BN < DOWN_BN ? BN : DOWN_BN) - 1) / (BN < DOWN_BN ? BN : DOWN_BN) : (P.N + BN_OUT - 1) / BN_OUT;
        P.tile_begin = total;
        P.readers = P.tiles_n;
        g.first_tile[i] = total;
        total += P.tiles_m * P.tiles_n;
        if (P.signal) g.n_lead = total;
        P.wait_need = (P.K1 + (BN < DOWN_BN ? BN : DOWN_BN) - 1) / (BN < DOWN_BN ? BN : DOWN_BN);   // column tiles of the producer, whose N is this problem's K1
    }
    g.total_tiles = total;
    if (total == 0) return SD_OK;
    // A few tiles of longer K loops behind the producers' (text keys / values in a q, k, v launch) are dealt round-robin like those: in
    // one XCD's range they held up its other tiles (7904x1920x640 with 20 text tiles: every XCD was done after 26 us, that one after 34).  How few makes
    // no difference that could be measured (two blocks, none / up to 6 / 12.5 / 25 / 50 % of the tiles: 2 x 3952 x 640 589 581 582 582 583, 2 x 1024 x 1280 + 64
    // 519 518 514 512 514, 4 x 1200 x 640 + 32 422 418 418 420 417).
    int front = 0;
    for (int i = 0; i < g.n && (g.p[i].signal || g.p[i].K0 > g.p[g.n - 1].K0); ++i) front = g.p[i].tile_begin + g.p[i].tiles_m * g.p[i].tiles_n;
    if (front - g.n_lead <= total / 8) g.n_lead = front;
    if (SD_DRY_RUN("gemm %dx%d/%d waves/%d stages%s%s%s%s%s; ", BM, BN, WGM * WGN, STAGES, GEGLU ? " geglu" : "", RES32 ? " res32" : "", guard ? " guard" : "",
                   !g.p[0].signal ? "" : g.p[0].nonce ? " records" : " flags", dry_detail(", %d problems", g.n)))
        return SD_OK;
    if (guard)
        hipLaunchKernelGGL((gemm_kernel<BM, BN, BK, WGM, WGN, STAGES, GEGLU, true, RES32>), dim3(g.n_lead + ((total - g.n_lead + 7) & ~7)), dim3(64 * WGM * WGN), 0, stream, g);
    else
        hipLaunchKernelGGL((gemm_kernel<BM, BN, BK, WGM, WGN, STAGES, GEGLU, false, RES32>), dim3(g.n_lead + ((total - g.n_lead + 7) & ~7)), dim3(64 * WGM * WGN), 0, stream, g);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

template <int BM, int BN, int BK, int WGM, int WGN, int STAGES>
static int launch_res(GemmGroup& g, const GemmChoice& c, hipStream_t stream) {
    if (c.res32) return launch_cfg<BM, BN, BK, WGM, WGN, STAGES, false, true>(g, c.guard, stream);
    return launch_cfg<BM, BN, BK, WGM, WGN, STAGES, false, false>(g, c.guard, stream);
}

// Which kernel, from the problems' sizes alone.
GemmChoice gemm_choice(const GemmGroup& g) {
    bool geglu = false;   // a GEGLU group: GEGLU problems plus, possibly, the plain down-projections they wait for
    bool guard = false;
    int maxN = 0;
    double lead = 0;      // down-projection tiles of 128 rows: workgroups too, ahead of the others
    double depth = 0;     // K, summed over those tiles
    long t128 = 0, t256 = 0;   // workgroup tiles of 128 and 256 rows x 128 output columns, down-projections aside
    int gM = 0, gF = 0, gK = 0, gr = 0;   // the GEGLU problems: rows in all, largest F, K and rank
    bool res32 = false;   // some problem adds an fp32 residual: take the kernel that prefetches it
    int n_main = 0;       // problems that are not down-projections
    bool mixed = false;   // ... of different widths or depths
    int N0 = 0, K0 = 0;
    for (int i = 0; i < g.n; ++i) {
        const GemmProblem& P = g.p[i];
        if (P.geglu_F > 0) geglu = true;
        if (P.Mp == 0 || P.N == 0) continue;
        if ((P.K0 & 63) || (P.K1 & 63)) guard = true;
        if (P.res && P.res_f32) res32 = true;
        if (P.N > maxN) maxN = P.N;
        if (P.signal) {
            lead += (double)((P.Mp + 127) / 128) * ((P.N + DOWN_BN - 1) / DOWN_BN);
            continue;
        }
        mixed = mixed || (n_main++ && (P.N != N0 || P.K0 != K0));
        N0 = P.N, K0 = P.K0;
        if (P.geglu_F > 0) {
            gM += P.Mp;
            gF = P.N > gF ? P.N : gF;
            gK = P.K0 > gK ? P.K0 : gK;
            gr = P.K1 > gr ? P.K1 : gr;
        }
        const long tiles = (long)((P.Mp + 127) / 128) * ((P.N + 127) / 128);
        t128 += tiles;
        t256 += (long)((P.Mp + 255) / 256) * ((P.N + 127) / 128);
        depth += (double)tiles * P.K0;
    }
    auto take = [&](GemmTiles t) { return GemmChoice{t, guard, res32}; };
    // Tile choice.  What a tile costs per 64 deep step is its operand bytes (a CU takes in 100-125 GB/s
    // from L2 whatever the ring depth) or its MFMAs, whichever is longer, and the launch takes as long
    // as its most loaded CU; so: the largest tiles that still give every CU the same number of them.
    // Times below are single projections of rank 64, us, measured on one machine.
    const double meanK = t128 ? depth / t128 : 0;
    // GEGLU: geglu_tiles (128 columns of W are 64 of the output)
    if (geglu) switch (geglu_tiles(gM, gF, gK, gr, false)) {
        case GEGLU_64x64_3STAGES: return take(GEMM_GEGLU_64x128_3STAGES);
        case GEGLU_64x64: return take(GEMM_GEGLU_64x128);
        case GEGLU_256x128: return take(GEMM_GEGLU_256x256);
        default: return take(GEMM_GEGLU_128x128);
        }
    // Down-projections (N = rank <= 64) alone: 64x64 tiles, 5-stage ring.
    if (maxN <= 64) return take(GEMM_64x64);
    if (t128 < 512) {
        // at most one 128x128 tile per CU, and most CUs have one: that tile with a deep ring, one
        // workgroup per CU (2048x1280x5120: 42.0, 53.7 with 64x128 tiles, of which 64 CUs get two)
        if (t128 > 128 && gemm_one_round(t128, (long)lead)) return take(GEMM_128x128_ONE_ROUND);
        // more than that (the down-projection's tiles count), but at most one of 256x128 per CU, and no short K loop: those
        // (8192x640x2560: 41.1, 48.2 with 128x128 tiles; 4757x1280x1280: 26.4, 33.1 with 64x128;
        // 6000x640x2560 34.5, 44.5 with 128x128 tiles; at K = 640 the ramps of the larger tile lose: 24.1 against 21.0)
        if (t128 > 128 && t256 + lead / 2 <= 256 && meanK >= 1024) return take(GEMM_256x128_ONE_ROUND);
        // few tiles: 64x128 spreads them over more CUs, two workgroups on a CU at most: three ring stages
        if (t128 <= 128) return take(GEMM_64x128_3STAGES);
        // up to three on a CU where the K loop is short (8192x640x640: 17.3, 18.3 with 128x128)
        if (t128 > 256 && meanK < 1024) return take(GEMM_64x128);
    }
    // One large plain projection with a long K loop (no launch of the transformer block: the
    // 8192 x 4096 x 4096 yardstick takes 220, 245 at 256x128, 260 at 128x128; 8192x8192x2048 + 64 256, 284, 290; but
    // 16384x1280x5120 + 64, five of these tiles wide, 254, 217, 236).  Not for grouped
    // launches: the q/k/v group with its short text-context problems loses a third.
    if (!res32 && n_main == 1 && t256 >= 512 && meanK >= 2048) return take(GEMM_256x256);
    // 128x128 tiles, two workgroups per CU.  Of eight 32x64 wavefronts where problems of different sizes share the launch (q, k,
    // v transposed, text keys): their tiles load the CUs unevenly, and one that has a CU to itself is faster with more
    // wavefronts (attention blocks, us, four / eight: 4 x 3952 tokens of 640 channels with text keys + 64 106.7 / 100.4, 2 x 988 of
    // 1280 + 16 85.6 / 79.8, 2 x 4096 of 320 + 8 109.8 / 100.5, 4 x 3952 of 640 + 32 275.4 / 279.2; 80 of them 0.91 to 1.014)
    if (mixed && !res32) return take(GEMM_128x128_8WAVES);
    // ... of four 64x64 otherwise (4757x1280x1280: 25.9, 33.1 with 64x128, 26.9 with eight wavefronts; the segments of a multi-adapter
    // call: 8 x 4096 of 640 channels 45.0 / 45.6, 2999,2221,1552,1847,895 of 1280 48.6 / 50.7, of 320 up to 12 % the other way)
    return take(GEMM_128x128);
}

int launch_gemm_group(GemmGroup& g, hipStream_t stream) {
    SD_REQUIRE(g.n >= 1 && g.n <= GEMM_MAX_PROBLEMS, SD_EINVAL, "gemm group: %d problems", g.n);
    bool geglu = false;
    for (int i = 0; i < g.n; ++i) geglu = geglu || g.p[i].geglu_F > 0;
    for (int i = 0; i < g.n; ++i) {
        const GemmProblem& P = g.p[i];
        SD_REQUIRE((P.geglu_F > 0) == geglu || P.signal, SD_EINVAL, "gemm group mixes GEGLU and plain problems");
        SD_REQUIRE(P.Mp >= 0 && P.N >= 0 && P.K0 > 0 && P.K0 % 8 == 0 && P.K1 >= 0 && P.K1 % 8 == 0, SD_EINVAL,
                   "gemm problem %d: bad sizes M=%d N=%d K0=%d K1=%d", i, P.Mp, P.N, P.K0, P.K1);
        SD_REQUIRE(P.p0 && P.q0 && P.y && (P.K1 == 0 || (P.p1 && P.q1)), SD_EINVAL, "gemm problem %d: null operand", i);
        SD_REQUIRE(P.ldp0 % 8 == 0 && P.ldq0 % 8 == 0 && (P.K1 == 0 || (P.ldp1 % 8 == 0 && P.ldq1 % 8 == 0)), SD_EINVAL,
                   "gemm problem %d: leading dimensions must be multiples of 8", i);
        // lane offsets inside a tile are 32-bit byte offsets
        const int64_t span = 256 + (P.geglu_F > 0 ? P.geglu_F : 0);
        SD_REQUIRE(P.ldp0 > 0 && P.ldq0 > 0 && P.ldp0 * 256 < (1ll << 31) && P.ldq0 * span < (1ll << 31) &&
                       (P.K1 == 0 || (P.ldp1 > 0 && P.ldq1 > 0 && P.ldp1 * 256 < (1ll << 31) && P.ldq1 * span < (1ll << 31))),
                   SD_EINVAL, "gemm problem %d: leading dimension out of range", i);
        if (P.signal) {
            SD_REQUIRE(i == 0 || g.p[i - 1].signal, SD_EINVAL, "gemm group: signalling problem %d after a plain one", i);
            SD_REQUIRE(!P.y_f32 && !P.res && !P.wait && P.N % 4 == 0 && P.ldy % 4 == 0 && P.geglu_F == 0, SD_EINVAL,
                       "gemm problem %d: a signalling problem stores plain bf16 rows", i);
        }
        SD_REQUIRE(!P.nonce || (P.signal ? P.N <= DEP_PRODUCERS * DOWN_BN : (P.wait && !P.wait_cols && P.K1 <= DEP_PRODUCERS * DOWN_BN)), SD_EINVAL,
                   "gemm problem %d: what a dependency record does not hold", i);
        SD_REQUIRE(!P.wait || (P.K1 > 0 && g.p[0].signal), SD_EINVAL, "gemm problem %d waits but the group has no producer", i);
    }
    // drop empty problems
    int w = 0;
    for (int i = 0; i < g.n; ++i)
        if (g.p[i].Mp > 0 && g.p[i].N > 0) { if (w != i) g.p[w] = g.p[i]; ++w; }
    g.n = w;
    if (w == 0) return SD_OK;
    const GemmChoice c = gemm_choice(g);
    switch (c.tiles) {
    case GEMM_GEGLU_64x128_3STAGES: return launch_cfg<64, 128, 64, 2, 2, 3, true, false>(g, c.guard, stream);
    case GEMM_GEGLU_64x128: return launch_cfg<64, 128, 64, 2, 2, 2, true, false>(g, c.guard, stream);
    case GEMM_GEGLU_256x256: return launch_cfg<256, 256, 64, 4, 2, 2, true, false>(g, c.guard, stream);
    case GEMM_GEGLU_128x128: return launch_cfg<128, 128, 64, 2, 2, 2, true, false>(g, c.guard, stream);
    case GEMM_64x64: return launch_cfg<64, 64, 64, 2, 2, 5, false, false>(g, c.guard, stream);
    case GEMM_128x128_ONE_ROUND: return launch_res<128, 128, 64, 4, 2, 4>(g, c, stream);
    case GEMM_256x128_ONE_ROUND: return launch_res<256, 128, 64, 4, 2, 3>(g, c, stream);
    case GEMM_64x128_3STAGES: return launch_res<64, 128, 64, 2, 2, 3>(g, c, stream);
    case GEMM_64x128: return launch_res<64, 128, 64, 2, 2, 2>(g, c, stream);
    case GEMM_256x256: return launch_cfg<256, 256, 64, 4, 2, 2, false, false>(g, c.guard, stream);
    case GEMM_128x128_8WAVES: return launch_cfg<128, 128, 64, 4, 2, 2, false, false>(g, c.guard, stream);
    default: return launch_res<128, 128, 64, 2, 2, 2>(g, c, stream);
    }
}

__global__ void clear_flags_kernel(int32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}
int launch_clear_flags(int32_t* p, int n, hipStream_t stream) {
    if (n <= 0 || SD_DRY_RUN("clear; ")) return SD_OK;
    hipLaunchKernelGGL(clear_flags_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, p, n);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}
int gemm_dep_timeouts(long long* count) {
    unsigned long long v = 0;
    SD_HIP_CHECK(hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_gemm_dep_timeouts), sizeof(v)));
    *count = (long long)v;
    return SD_OK;
}

}  // namespace sd
