// From self-attention's output to the feed-forward's input in one launch, for blocks of 320 and 640 channels: output projection
// and residual, LayerNorm, cross-attention query, cross-attention over the text keys, its output projection and
// residual, LayerNorm.  A workgroup takes 32 rows through all of it; the rows never leave the CU, the residual stays in registers.
//
// What bounds it: the weights, and the phases between them.  Every workgroup reads all of them, and 256 CUs take one and the same matrix out of L2
// at 107-116 GB/s each (whole 128-byte lines straight into LDS; 16 rows of 64 bytes a load come in at 65, and fragments loaded
// straight into registers at 37, because an instruction's adjacent lanes then lie in different lines): 7.1 us for 640 x 640.  A step's clocks at 7904
// rows: half in the three products, 13 % in cross-attention, 12 % in the LayerNorms, the rest first operands, residual and stores.  Over the whole
// launch, at 8192 rows + 64, the matrix cores are busy for 18 % of the time, the vector ALU for 21, LDS reads for 25, of which bank conflicts are 27.
// us a launch, kernel traces of the same stacks one behind the other, the six launches that it stands for (output projection, LayerNorm, query,
// attention, output projection, LayerNorm) / here: 8192 rows of 640 channels + 64 80.1 (19.8, 6.7, 16.3, 10.7, 19.8, 6.7) / 56.5 (58.6 where weights come from
// HBM), 7904 without adapter 69.7 / 51.0; 8192 rows of 320 + 16 49.5 / 31.4, 2688 34.4 / 28.0.
//
// Wavefront w owns columns 64 w .. 64 w + 63 of every product, which are also attention head w: the query it computes is the one
// it needs, and the output it computes is its part of the next operand.  What it needs of the weights nobody else does, so
// each wavefront has a slot of its own in LDS, fed in order of use without barriers and over the products' edges.  Barriers
// remain where rows change hands: one to see t = x A^T, one before and one after the operand tile is rewritten, one per LayerNorm.
#include "gemm_dma.hpp"
#include "read_ahead.hpp"

namespace sd {

constexpr int CHAIN_ROWS = 32, CHAIN_RANK = 128, CHAIN_KEYS = 80;

struct ChainProj { const uint16_t *W, *A, *B, *bias; int32_t r; float scale; };
struct ChainArgs {
    const uint16_t* a;          // self-attention's output [Bn * T, C]
    const float* h_in; float* h;// the residual stream before and after [Bn * T, C]
    uint16_t* n;                // the feed-forward's input [Bn * T, C]
    const uint16_t *k, *vt;     // text keys [Bn * Tc, C], values [C, Bn * Tkp]
    ChainProj o1, q2, o2;
    const uint16_t *g2, *b2, *g3, *b3;
    int64_t ldvt;
    int32_t T, Tc, Tkp;
    float eps, kscale;          // the scores' factor to exponents of 2 (1: it is in the keys)
};

template <int V> using IntC = std::integral_constant<int, V>;

template <int HEADS>
struct Chain {
    static constexpr int NW = HEADS, C = 64 * HEADS;
    static constexpr int XP = C / 8 + 1;                       // 16-byte chunks of an operand row, one of them padding (odd: rows 16 apart in no bank)
    static constexpr int TP = CHAIN_RANK / 8 + 1;              // ... of a row of t
    static constexpr int NCONST = 7;                           // biases and affines, as fp32
    static constexpr int SLOT = 512;                           // chunks of an item of the stream: 64 rows of 128 bytes
    static constexpr int X = 0, T = X + CHAIN_ROWS * XP, STATS = T + CHAIN_ROWS * TP, CONSTS = STATS + CHAIN_ROWS * NW / 2,
                         RING = CONSTS + NCONST * C / 4;
    static constexpr int LDS_CH = RING + NW * SLOT;
    static constexpr int AQ = (HEADS + 3) / 4;                 // items of 16 rows of A, four 64 deep k-steps each
    static_assert(LDS_CH <= 160 * 64 && (HEADS > 5 || LDS_CH <= 80 * 64), "LDS: of five wavefronts, two workgroups");
};

__device__ __forceinline__ float quad_rows_sum(float v) {      // over the four rows of 16 lanes, in every lane
    float a = v, b = v;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    float lo, hi;
    both_halves(a + b, lo, hi);
    return lo + hi;
}
__device__ __forceinline__ float quad_rows_max(float v) {
    float a = v, b = v;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    float lo, hi;
    both_halves(fmaxf(a, b), lo, hi);
    return fmaxf(lo, hi);
}

template <int HEADS, bool AHEAD>
__global__ __launch_bounds__(64 * HEADS, 3) void chain_kernel(const ChainArgs g, const std::conditional_t<AHEAD, ReadRanges, NoRanges> ra) {
    using K = Chain<HEADS>;
    constexpr int NW = K::NW, C = K::C, XP = K::XP, TP = K::TP, SLOT = K::SLOT, AQ = K::AQ;
    __shared__ u32x4 lds[K::LDS_CH];

    // the argument words' cache lines in one round of scalar loads: left to their uses they would come one after the other
    {
        const uint32_t* const w = reinterpret_cast<const uint32_t*>(&g);
        static_assert(sizeof(ChainArgs) <= 256, "four lines");
        asm volatile("" ::"s"(w[0]), "s"(w[16]), "s"(w[32]), "s"(w[48]));
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int sample = blockIdx.y, row0 = blockIdx.x * CHAIN_ROWS;
    const int last = min(CHAIN_ROWS, g.T - row0) - 1;          // the block's last row that is there: those past it repeat it and are not stored
    const int64_t first = (int64_t)sample * g.T + row0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    const int slot = K::RING + wave * SLOT;
    const uint32_t to = lds0 + slot * 16;

    // ---- the stream: everything this wavefront reads of the weights and more, 8 KB an item, in order of use
    // The three products' parts in turn, and of the part at hand: items left, where the next begins.  The residual comes amidst
    // the first product, whose steps hide its way from HBM; the text keys and values follow the second.
    enum { PART_A, PART_W, PART_RES, PART_W2, PART_B, PART_KV, PARTS };
    int part = -1, kind = 0, left = 0, rank = 0;
    const char* from = nullptr;
    constexpr int HALF = HEADS / 2;
    constexpr int END = 2 * PARTS + PART_KV;
    const uint32_t weven = (lane >> 3) * (C * 2) + ((lane & 7) ^ (lane >> 4)) * 16;
    auto enter = [&]() __attribute__((always_inline)) {
        do {
            ++part;
            const int p = part / PARTS, at = part - p * PARTS;
            // (field by field: a reference into the arguments would put them into scratch memory)
            if (at == PART_A) {
                rank = p == 0 ? g.o1.r : p == 1 ? g.q2.r : g.o2.r;
                from = reinterpret_cast<const char*>(p == 0 ? g.o1.A : p == 1 ? g.q2.A : g.o2.A);
                const int tiles = (rank + 15) / 16;
                left = tiles > wave ? (tiles - wave + NW - 1) / NW * AQ : 0;
            } else if (at == PART_W) {
                from = reinterpret_cast<const char*>((p == 0 ? g.o1.W : p == 1 ? g.q2.W : g.o2.W) + (int64_t)wave * 64 * C);
                left = HALF;
            } else if (at == PART_RES) {
                left = p == 0 ? 1 : 0;
            } else if (at == PART_W2) {
                left = HEADS - HALF;
            } else if (at == PART_B) {
                from = reinterpret_cast<const char*>((p == 0 ? g.o1.B : p == 1 ? g.q2.B : g.o2.B) + (int64_t)wave * 64 * rank);
                left = (rank + 63) / 64;
            } else {
                left = p == 1 ? 3 : 0;
            }
            kind = at;
        } while (left == 0 && part < END);
    };
    // the next item's loads.  kinds: what it can be at this place
    enum { A_ = 1, W_ = 2, B_ = 4, RES_ = 8, K0_ = 16, K1_ = 32, V0_ = 64 };
    auto issue = [&](auto kinds) __attribute__((always_inline)) {
        constexpr int KINDS = decltype(kinds)::value;
        if (!(KINDS & (K1_ | V0_)) && left == 0 && part < END) enter();
        --left;
        if (part == END) return;
        if ((KINDS & W_) && (KINDS == W_ || kind == PART_W || kind == PART_W2)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) dma16_so(from + j * 8 * (C * 2), j & 1 ? weven ^ 64 : weven, to + j * 1024);
            from += 128;
            return;
        }
        int ln = lane;
        asm volatile("" : "+v"(ln));    // the addresses are formed here: kept over the loops they would fill the registers
        const int r8 = ln >> 3, sw = ((ln & 7) ^ (ln >> 4)) * 16;   // odd kilobytes of a slot: sw ^ 64
        if ((KINDS & A_) && kind == PART_A) {
            const int tiles = (rank + 15) / 16, all = (tiles - wave + NW - 1) / NW * AQ, item = all - left - 1;
            const int at = wave + (item / AQ) * NW, q = item % AQ;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int row = min(at * 16 + (j & 1) * 8 + r8, rank - 1), ks = min(q * 4 + j / 2, HEADS - 1);
                dma16_so(from + ks * 128, (uint32_t)(row * (C * 2) + (sw ^ (j & 1 ? 64 : 0))), to + j * 1024);
            }
        } else if ((KINDS & B_) && kind == PART_B) {
            const int at = ((rank + 63) / 64 - left - 1) * 128;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = at + (sw ^ (j & 1 ? 64 : 0));
                const void* src = from + (j * 8 + r8) * rank * 2 + c;
                if (c >= 2 * rank) src = g_gemm_zeros;
                dma16(src, to + j * 1024);
            }
        } else if ((KINDS & RES_) && kind == PART_RES) {
            // the residual: 32 rows of 256 bytes, chunk c of row r at c ^ (r % 16)
            const char* const base = reinterpret_cast<const char*>(g.h_in + first * C + wave * 64);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int row = j * 4 + (ln >> 4);
                dma16_so(base, (uint32_t)(min(row, last) * (C * 4) + ((ln ^ row) & 15) * 16), to + j * 1024);
            }
        } else {
            // text keys 0 .. 63; keys and values 64 .. 79; values 0 .. 63
            const uint16_t* const kb = g.k + (int64_t)sample * g.Tc * C + wave * 64;
            const uint16_t* const vb = g.vt + (int64_t)wave * 64 * g.ldvt + (int64_t)sample * g.Tkp;
            if (KINDS & K0_) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    dma16_so(kb, (uint32_t)(min(j * 8 + r8, g.Tc - 1) * (C * 2) + (sw ^ (j & 1 ? 64 : 0))), to + j * 1024);
            } else if (KINDS & K1_) {
                // as rows of K, then as 32 bytes of each row of V^T
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (j < 2) {
                        dma16_so(kb, (uint32_t)(min(64 + j * 8 + r8, g.Tc - 1) * (C * 2) + (sw ^ (j & 1 ? 64 : 0))), to + j * 1024);
                    } else {
                        const int d = ((j & 1) * 64 + ln) >> 1, key = 64 + (ln & 1) * 8;
                        const void* src = vb + d * g.ldvt + key;
                        if (key >= g.Tkp) src = g_gemm_zeros;
                        dma16(src, to + j * 1024);
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int c = sw ^ (j & 1 ? 64 : 0);
                    const void* src = reinterpret_cast<const char*>(vb + (j * 8 + r8) * g.ldvt) + c;
                    if (c >= 2 * g.Tkp) src = g_gemm_zeros;
                    dma16(src, to + j * 1024);
                }
            }
        }
    };
    // the item at hand has landed
    auto take = [&]() __attribute__((always_inline)) { wait_vmcnt<0>(); };
    // its contents are in registers: the slot takes the next one
    auto release = [&](auto kinds) __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        issue(kinds);
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- operand rows and constants
    {
        u32x4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ch = tid + i * C, row = ch / (C / 8), c = ch - row * (C / 8);
            v[i] = *as_global(reinterpret_cast<const u32x4*>(g.a + (first + min(row, last)) * C + c * 8));
        }
        const uint16_t* const src[K::NCONST] = {g.o1.bias, g.q2.bias, g.o2.bias, g.g2, g.b2, g.g3, g.b3};
        uint16_t cv[K::NCONST];
#pragma unroll
        for (int i = 0; i < K::NCONST; ++i) cv[i] = *as_global((src[i] ? src[i] : reinterpret_cast<const uint16_t*>(g_gemm_zeros)) + (src[i] ? tid : 0));
        issue(IntC<A_ | W_>());
        float* const consts = reinterpret_cast<float*>(lds + K::CONSTS);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ch = tid + i * C, row = ch / (C / 8), c = ch - row * (C / 8);
            lds[K::X + row * XP + c] = v[i];
        }
#pragma unroll
        for (int i = 0; i < K::NCONST; ++i) consts[i * C + tid] = bf16_to_f32(cv[i]);
    }
    __syncthreads();

    // a value the compiler takes for a new one: what is formed from it is formed where it is used, and not kept in registers over the loops
    auto fresh = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    const int lsw = (l16 >> 1) & 7;
    // (chunk indices: pointers that a loop chooses between lose their address space, and flat loads wait for the stream)
    const int xrow = K::X + l16 * XP + quad, trow = K::T + l16 * TP + quad;
    // four columns' values of a bias or affine
    auto cst = [&](int qd, int which, int ni) { return __builtin_bit_cast(f32x4, lds[K::CONSTS + which * (C / 4) + wave * 16 + ni * 4 + qd]); };
    enum { K_BO1, K_BQ2, K_BO2, K_G2, K_B2, K_G3, K_B3 };

    // a 64 deep k-step of the product with 64 rows of a slot: acc += x rows (LDS, at x) * rows of the slot
    f32x4 acc[2][4], h[2][4];     // h: the residual stream
    auto clear = [&]() {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto step = [&](int x, int next) __attribute__((always_inline)) {    // next: chunks to the row 16 further on
        bf16x8 xf[2][2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            xf[kk][0] = __builtin_bit_cast(bf16x8, lds[x + kk * 4]);
            xf[kk][1] = __builtin_bit_cast(bf16x8, lds[x + next + kk * 4]);
        }
        bf16x8 wf[2][4];
        take();
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) wf[kk][ni] = __builtin_bit_cast(bf16x8, lds[slot + (ni * 16 + l16) * 8 + ((kk * 4 + quad) ^ lsw)]);
        release(IntC<A_ | W_ | B_ | RES_ | K0_>());
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni)
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[kk][ni], xf[kk][mi], acc[mi][ni], 0, 0, 0);
    };
    // acc = x W^T + (scale x A^T) B^T for this wavefront's columns; everyone has read x when it returns
    auto project = [&](int r, float scale, int which) __attribute__((always_inline)) {
#pragma unroll 1
        for (int at = wave; at * 16 < ((r + 63) & ~63); at += NW) {
            f32x4 t[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
            if (at * 16 < r)
#pragma unroll 1
                for (int q = 0; q < AQ; ++q) {
                    bf16x8 af[4][2];
                    const u32x4* const w = lds + slot + l16 * 8;
                    take();
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int kk = 0; kk < 2; ++kk) af[s][kk] = __builtin_bit_cast(bf16x8, w[s * 128 + ((kk * 4 + quad) ^ lsw)]);
                    release(IntC<A_ | W_>());
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        if (q * 4 + s < HEADS)
#pragma unroll
                            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                                for (int mi = 0; mi < 2; ++mi) {
                                    const bf16x8 xf = __builtin_bit_cast(bf16x8, lds[xrow + mi * 16 * XP + (q * 4 + s) * 8 + kk * 4]);
                                    t[mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[s][kk], xf, t[mi], 0, 0, 0);
                                }
                }
            const int col = at * 16 + quad * 4;
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)(col + e < r ? t[mi][e] * scale : 0.f);
                *reinterpret_cast<bf16x4*>(reinterpret_cast<uint16_t*>(lds + K::T + (mi * 16 + l16) * TP) + col) = o;
            }
        }
        clear();
        int x = xrow, xt = trow, steps = HALF, next = 16 * XP;
        asm volatile("" : "+v"(x), "+v"(xt));
#pragma unroll 1
        for (int part = 0; part < 3; ++part) {
#pragma unroll 1
            for (; steps > 0; --steps, x += 8) step(x, next);
            if (part == 0) {
                if (which == 0) {
                    const int ln = fresh(lane), lr = ln & 15, qd = ln >> 4;
                    const u32x4* const rs = lds + slot;
                    take();
#pragma unroll
                    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                        for (int ni = 0; ni < 4; ++ni) h[mi][ni] = __builtin_bit_cast(f32x4, rs[(mi * 16 + lr) * 16 + ((ni * 4 + qd) ^ lr)]);
                    release(IntC<W_>());
                }
                steps = HEADS - HALF;
            } else if (part == 1) {
                __syncthreads();
                x = xt;
                next = 16 * TP;
                steps = (r + 63) / 64;
            }
        }
    };
    auto store_x = [&](int lr, int qd, int mi, int ni, const f32x4& v) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)v[e];
        *reinterpret_cast<bf16x4*>(reinterpret_cast<uint16_t*>(lds + K::X + (mi * 16 + lr) * XP) + wave * 64 + ni * 16 + qd * 4) = o;
    };
    // LayerNorm of h: each wavefront's mean and squares about it over its 64 columns, then all of them together
    auto layernorm = [&](int kg, int kb, auto put) {
        const int ln = fresh(lane), lr = ln & 15, qd = ln >> 4;
        u32x2* const stats = reinterpret_cast<u32x2*>(lds + K::STATS);
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            float s = 0.f;
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) s += (h[mi][ni][0] + h[mi][ni][1]) + (h[mi][ni][2] + h[mi][ni][3]);
            const float mean = quad_rows_sum(s) * (1.0f / 64);
            float q = 0.f;
#pragma unroll
            for (int ni = 0; ni < 4; ++ni)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d = h[mi][ni][e] - mean;
                    q = fmaf(d, d, q);
                }
            q = quad_rows_sum(q);
            if (qd == 0) stats[(mi * 16 + lr) * NW + wave] = u32x2{__float_as_uint(mean), __float_as_uint(q)};
        }
        __syncthreads();
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            // (each row of 16 lanes adds up every fourth wavefront's)
            constexpr int EACH = (NW + 3) / 4;
            u32x2 st[EACH];
            float mean = 0.f, q = 0.f;
#pragma unroll
            for (int i = 0; i < EACH; ++i) {
                st[i] = stats[(mi * 16 + lr) * NW + min(i * 4 + qd, NW - 1)];
                mean += i * 4 + qd < NW ? __uint_as_float(st[i][0]) : 0.f;
            }
            mean = quad_rows_sum(mean) * (1.0f / NW);
#pragma unroll
            for (int i = 0; i < EACH; ++i) {
                const float d = __uint_as_float(st[i][0]) - mean;
                q += i * 4 + qd < NW ? fmaf(64.f * d, d, __uint_as_float(st[i][1])) : 0.f;
            }
            q = quad_rows_sum(q);
            const float rstd = rsqrtf(q * (1.0f / C) + g.eps);
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) {
                const f32x4 gm = cst(qd, kg, ni), bt = cst(qd, kb, ni);
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (h[mi][ni][e] - mean) * rstd * gm[e] + bt[e];
                put(lr, qd, mi, ni, v);
            }
        }
    };

    // ---- the three projections: one body, so that the code stays small
#pragma unroll 1
    for (int which = 0; which < 3; ++which) {
        project(which == 0 ? g.o1.r : which == 1 ? g.q2.r : g.o2.r, which == 0 ? g.o1.scale : which == 1 ? g.q2.scale : g.o2.scale, which);
        if (which == 0) {
            // the residual, LayerNorm
            const int qd = fresh(lane) >> 4;
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 4; ++ni) h[mi][ni] = (acc[mi][ni] + cst(qd, K_BO1, ni)) + h[mi][ni];
            layernorm(K_G2, K_B2, store_x);
            __syncthreads();
        } else if (which == 1) {
            const int ln = fresh(lane), lr = ln & 15, qd = ln >> 4, ls = (lr >> 1) & 7;
            // the query of cross-attention, in the order of the MFMA's second operand: a lane has four columns of one block of
            // 16 and four of the next for each k-step, and the keys are read in that order
            bf16x8 qf[2][2];
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 4; ++ni) {
                    const f32x4 b = cst(qd, K_BQ2, ni);
#pragma unroll
                    for (int e = 0; e < 4; ++e) qf[mi][ni >> 1][(ni & 1) * 4 + e] = (__bf16)(acc[mi][ni][e] + b[e]);
                }
            {
                // scores: lane lr is the row, its keys are kt * 16 + qd * 4 + e.  Keys past the last one, which are that one again, start at
                // -inf and stay there (a finite start is lost in the rounding of scores of 1e37 and above; where the product is inf or NaN, so is a real key's)
                f32x4 s[2][5];
                auto key_frag = [&](const u32x4* rows, int kk) {     // 16 keys, rows of 128 bytes
                    const u32x2* const k8 = reinterpret_cast<const u32x2*>(rows + lr * 8);
                    const int c = kk * 4 + (qd >> 1);
                    const u32x2 lo = k8[(c ^ ls) * 2 + (qd & 1)], hi = k8[((c + 2) ^ ls) * 2 + (qd & 1)];
                    return __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
                };
                {
                    const u32x4* const ks = lds + slot;
                    take();
                    bf16x8 kf[4][2];
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                        for (int kk = 0; kk < 2; ++kk) kf[kt][kk] = key_frag(ks + kt * 128, kk);
                    release(IntC<K1_>());
#pragma unroll
                    for (int kt = 0; kt < 5; ++kt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) s[0][kt][e] = s[1][kt][e] = kt * 16 + e < g.Tc - qd * 4 ? 0.f : -INFINITY;
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                            for (int mi = 0; mi < 2; ++mi) s[mi][kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kt][kk], qf[mi][kk], s[mi][kt], 0, 0, 0);
                }
                // values past the last key, in its group of eight, are anyone's: zeros, as 0 * NaN is none.  (A lane mends one row of V^T)
                auto mend = [&](int at) {
                    const int n = g.Tc & 7;
                    u32x4 v = lds[at];
#pragma unroll
                    for (int w = 0; w < 4; ++w) v[w] &= 2 * w + 1 < n ? 0xffffffffu : 2 * w < n ? 0xffffu : 0u;
                    lds[at] = v;
                };
                u32x2 v1[4];
                {
                    take();
                    const u32x4* const ks = lds + slot;
                    const bf16x8 kf[2] = {key_frag(ks, 0), key_frag(ks, 1)};
                    if (g.Tc > 64 && (g.Tc & 7)) mend(slot + 128 + ln * 2 + ((g.Tc - 64) >> 3));
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) v1[dt] = reinterpret_cast<const u32x2*>(ks + 128)[(dt * 16 + lr) * 4 + qd];
                    release(IntC<V0_>());
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                        for (int mi = 0; mi < 2; ++mi) s[mi][4] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kk], qf[mi][kk], s[mi][4], 0, 0, 0);
                }
                // probabilities.  The sum adds the rounded values, which are what is multiplied
                bf16x8 pf[2][3];
                float inv[2];
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) {
                    if (g.kscale != 1.0f)
#pragma unroll
                        for (int kt = 0; kt < 5; ++kt) s[mi][kt] *= g.kscale;
                    float m = s[mi][0][0];
#pragma unroll
                    for (int i = 1; i < 20; ++i) m = fmaxf(m, s[mi][i / 4][i % 4]);
                    m = quad_rows_max(m);
                    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
                    float l[2] = {0.f, 0.f};
#pragma unroll
                    for (int i = 0; i < 10; ++i) {
                        const bf16x2 p = {(__bf16)__builtin_amdgcn_exp2f(s[mi][i / 2][i % 2 * 2] - m), (__bf16)__builtin_amdgcn_exp2f(s[mi][i / 2][i % 2 * 2 + 1] - m)};
                        pf[mi][i / 4][i % 4 * 2] = p[0];
                        pf[mi][i / 4][i % 4 * 2 + 1] = p[1];
                        l[i & 1] = __builtin_amdgcn_fdot2_f32_bf16(p, ones, l[i & 1], false);
                    }
#pragma unroll
                    for (int e = 4; e < 8; ++e) pf[mi][2][e] = (__bf16)0.f;
                    inv[mi] = 1.0f / quad_rows_sum(l[0] + l[1]);
                }
                take();
                if (g.Tc < 64 && (g.Tc & 7)) mend(slot + ln * 8 + ((g.Tc >> 3) ^ ((ln >> 1) & 7)));
                const u32x2* const vs = reinterpret_cast<const u32x2*>(lds + slot);
                bf16x8 vf[4][2];
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int c = j * 4 + (qd >> 1), row = (dt * 16 + lr) * 8;
                        const u32x2 lo = vs[(row + (c ^ ls)) * 2 + (qd & 1)], hi = vs[(row + ((c + 2) ^ ls)) * 2 + (qd & 1)];
                        vf[dt][j] = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
                    }
                release(IntC<A_ | W_>());
                f32x4 o[2][4];
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                        for (int mi = 0; mi < 2; ++mi) {
                            if (j == 0) o[mi][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
                            const bf16x8 v = j < 2 ? vf[dt][j] : __builtin_bit_cast(bf16x8, u32x4{v1[dt][0], v1[dt][1], 0u, 0u});
                            o[mi][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pf[mi][j], o[mi][dt], 0, 0, 0);
                        }
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) store_x(lr, qd, mi, dt, o[mi][dt] * inv[mi]);
            }
            __syncthreads();
        }
    }
    // ---- the residual, LayerNorm
    const int ln = fresh(lane), lr = ln & 15, qd = ln >> 4, ls = (lr >> 1) & 7;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) h[mi][ni] = (acc[mi][ni] + cst(qd, K_BO2, ni)) + h[mi][ni];
    // out through this wavefront's ring, which is empty now, as rows of 256 bytes (the stream) and 128 (the normalised rows)
    u32x4* const out = lds + slot;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) out[(mi * 16 + lr) * 16 + ((ni * 4 + qd) ^ lr)] = __builtin_bit_cast(u32x4, h[mi][ni]);
    {
        float* const base = g.h + first * C + wave * 64;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int row = j * 4 + qd;
            const u32x4 v = out[row * 16 + ((ln ^ row) & 15)];
            if (row <= last) *as_global(reinterpret_cast<u32x4*>(base + (int64_t)row * C + lr * 4)) = v;
        }
    }
    layernorm(K_G3, K_B3, [&](int lr, int qd, int mi, int ni, const f32x4& v) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)v[e];
        const int row = mi * 16 + lr, c = ni * 2 + (qd >> 1);
        reinterpret_cast<bf16x4*>(out)[(row * 8 + (c ^ ls)) * 2 + (qd & 1)] = o;
    });
    {
        uint16_t* const base = g.n + first * C + wave * 64;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = j * 8 + (ln >> 3), c = ln & 7;
            const u32x4 v = out[row * 8 + (c ^ ((row >> 1) & 7))];
            if (row <= last) *as_global(reinterpret_cast<u32x4*>(base + (int64_t)row * C + c * 8)) = v;
        }
    }
    // (by the workgroups themselves: one behind them would wait for a CU's LDS)
    if constexpr (AHEAD)
        if (tid < 256) read_ahead<8>(ra, (int)(blockIdx.y * gridDim.x + blockIdx.x), tid);
}

// One workgroup of 640 channels fills a CU and takes 51 us (57 with adapters of rank 64) whatever the others do; the launches it stands for take
// their time by the row.  us of a one-block stack, launches / chain, by blocks of rows: 32 113 / 123, 63 141 / 147, 94 190 / 188 (+ 64 200 / 194),
// 126 196 / 192 (208 / 198), 164 250 / 238, 208 293 / 277 (310 / 287), 256 333 / 315 (348 / 325); in a second round, 288 351 / 364 (379 / 387),
// 512 653 / 646 (686 / 670).  So: one round that is a third full, or several whose last is nearly full, counted in rows: blocks that samples of odd lengths
// leave partly empty take as long as full ones (45 x 33 tokens + 16 278 / 286, 60 x 33 222 / 227; two rounds, 245 x 33 + 16 1191 / 1213, 250 x 40 + 128
// 1326 / 1336, 250 x 57 + 64 1402 / 1380; of 320 channels 180 x 33 + 64 725 / 728, 300 x 8 + 64 1061 / 1072, 300 x 75 + 128 1474 / 1501).  Without adapters
// the launches are in-tile projections of one round, and the line is later: 1 x 2880 183 / 187, 30 x 75 185 / 188, 60 x 48 253 / 255, 1 x 3264 208 / 204.
//   Of 320 channels two workgroups share a CU, which is a round of 512, and alone on a CU one is faster: up to 256 blocks 16 + 8 69.0 / 71.0,
// 26 + 8 74.7 / 78.6, 38 + 8 88.1 / 88.9, + 64 96 / 92, 64 + 8 104 / 99, 126 + 8 134 / 125, 256 205 / 187.  Past that without adapter, + 16, + 64, + 128, another
// machine: 268 199 / 199, 223 / 223, 223 / 225, 243 / 241; 308 219 / 218, 245 / 243, 244 / 247, 261 / 260; 348 234 / 228, 257 / 256, 258 / 256, 273 / 270; 444 271 / 262,
// 298 / 288, 298 / 291, 316 / 308; 496 291 / 278, 312 / 303, 310 / 304, 332 / 323 (the first machine's up to 440 blocks lay 1 % either way of these); in a
// second round 516 344 / 341, 376 / 370, 369 / 373, 385 / 399; 564 332 / 329, 369 / 360, 363 / 363, 383 / 392; 600 342 / 337, 379 / 367, 373 / 370, 389 / 398; 750
// 475 / 454, 524 / 489, 517 / 498, 541 / 528; 880 533 / 529, 585 / 567, 563 / 561, 587 / 600; in a third 1030 591 / 595, 643 / 635, 620 / 635, 658 / 682;
// 1352 834 / 840, 896 / 892, 876 / 891, 920 / 948 (+ 40 as + 16; + 96 380 / 386 at 516, in between elsewhere).  Not where the rows past a multiple of 8192 are not there, so that
// the launches need a round less: 86 x 95 tokens, 258 blocks, 266 / 271, 452 / 460, 435 / 444, 475 / 476; 6 x 2730, 516 blocks, 287 / 295, 311 / 327, 310 / 330, 339 / 359.
bool chain_takes(int Bn, int T, int C, int Tc, const sd_proj& o1, const sd_proj& q2, const sd_proj& o2) {
    const int rank = std::max(o1.r, std::max(q2.r, o2.r));
    if (Tc > CHAIN_KEYS || rank > CHAIN_RANK || Bn > 65535) return false;
    const long blocks = (long)Bn * ((T + CHAIN_ROWS - 1) / CHAIN_ROWS), rounds = (blocks + 255) / 256, rows = (long)Bn * T;
    const bool full = rows >= blocks * 28;
    if (C == 320) {
        if (blocks <= 256) return blocks >= 38;
        if (!full || rows <= 8192 * (rounds - 1)) return false;
        return blocks <= 512 || rank <= 40 || (rank <= 96 && blocks >= 600 && blocks <= 1024);
    }
    return C == 640 && (rounds == 1 ? rows >= (rank == 0 ? 3264 : 2880) : full && blocks >= 256 * rounds - 24);
}

int launch_chain(const ChainCall& c, hipStream_t stream, ReadAhead* ahead) {
    ChainArgs g;
    auto proj = [](const sd_proj& p) { return ChainProj{p.W, p.A, p.B, p.bias, p.r, p.scale}; };
    g.a = c.a; g.h_in = c.h; g.h = c.h; g.n = c.n; g.k = c.k; g.vt = c.vt;
    g.o1 = proj(*c.o1); g.q2 = proj(*c.q2); g.o2 = proj(*c.o2);
    g.g2 = c.g2; g.b2 = c.b2; g.g3 = c.g3; g.b3 = c.b3;
    g.Tkp = (c.Tc + 7) & ~7;
    g.ldvt = (int64_t)c.Bn * g.Tkp;
    g.T = c.T; g.Tc = c.Tc;
    g.eps = c.eps;
    g.kscale = c.k_prescaled ? 1.0f : ATTN_KSCALE;
    const dim3 grid((c.T + CHAIN_ROWS - 1) / CHAIN_ROWS, c.Bn);
    const ReadRanges ra = ahead ? ahead->take(8ull << 20, (long)grid.x * grid.y, 8) : ReadRanges{};
    if (SD_DRY_RUN("projection of the chain; layernorm of the chain; projection of the chain; attention of the chain; projection of the chain; layernorm of the chain%s; ",
                   dry_ranges(ra)))
        return SD_OK;
    auto launch = [&](auto heads) {
        constexpr int H = decltype(heads)::value;
        if (ra.n) hipLaunchKernelGGL((chain_kernel<H, true>), grid, dim3(64 * H), 0, stream, g, ra);
        else hipLaunchKernelGGL((chain_kernel<H, false>), grid, dim3(64 * H), 0, stream, g, NoRanges{});
    };
    if (c.C == 320) launch(IntC<5>());
    else launch(IntC<10>());
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

}  // namespace sd
