// What the GEMM kernels share: direct global -> LDS loads, their wait counts, GELU, and how a
// workgroup finds its tile.
#pragma once
#include "common.hpp"

namespace sd {

// XOR swizzle of the 16-byte chunk index inside an LDS row of CPR chunks (8: 128-byte rows,
// 4: 64-byte rows): any 16 consecutive rows put the same logical chunk in 16 distinct
// 16-byte slots of a 256-byte bank window.
template <int CPR>
__device__ __forceinline__ int swz(int row, int chunk) {
    return CPR == 8 ? (chunk ^ ((row >> 1) & 7)) : (chunk ^ ((row >> 2) & 3));
}

// GELU, exact (erf) form, with erf by Abramowitz & Stegun 7.1.26 (|error| <= 1.5e-7, far below
// bf16 resolution): erf(|x|) = 1 - (a1 t + ... + a5 t^5) exp(-x^2), t = 1 / (1 + p |x|).
// With x = z / sqrt(2) and h = z / 2:  gelu(z) = h (1 + erf(x)) = h + |h| erf(|x|), because erf is
// odd and h has the sign of x: no sign transfer, and sqrt(1/2) folds into the constants.
__device__ __forceinline__ float gelu_erf(float z) {
    const float az = fabsf(z);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752440f, az, 1.0f));
    float p = fmaf(1.061405429f, t, -1.453152027f);
    p = fmaf(p, t, 1.421413741f);
    p = fmaf(p, t, -0.284496736f);
    p = fmaf(p, t, 0.254829592f);
    p *= t;
    const float e = __builtin_amdgcn_exp2f((-0.5f * 1.44269504088896340736f * z) * z);
    const float r = fmaf(-p, e, 1.0f);          // erf(|x|) in [0, 1]
    const float h = 0.5f * z;
    return fmaf(fabsf(h), r, h);
}

// 256 bytes of zeros: where the lanes of a direct-to-LDS load point when their chunk lies
// past the end of a K segment (the load itself cannot zero-fill)
static __device__ __attribute__((aligned(256))) uint32_t g_gemm_zeros[64];

// One direct global -> LDS load: every lane fetches 16 bytes from its own global address and
// the wavefront's 64 pieces land contiguously at LDS byte address `lds_base` (wave-uniform).
// Written as inline assembly so that the compiler does not serialise the LDS reads of the
// tile being multiplied behind loads that target another ring stage; completion is tracked
// by hand with vmcnt (loads retire in order) and a workgroup barrier.
// DEV: the load is of device scope (it must observe data that a workgroup on another XCD, with
// its own L2, wrote during this launch with device-scope stores).
template <bool DEV = false>
__device__ __forceinline__ void dma16(const void* gptr, uint32_t lds_base) {
    if (DEV)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off sc1" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(gptr) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(gptr) : "memory", "m0");
}
// Same with a wave-uniform 64-bit base and a 32-bit unsigned byte offset per lane, which
// keeps the per-step address arithmetic on the scalar unit.
template <bool DEV = false>
__device__ __forceinline__ void dma16_so(const void* sbase, uint32_t voff, uint32_t lds_base) {
    if (DEV)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 sc1" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(voff), "s"(uniform_ptr(sbase)) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(voff), "s"(uniform_ptr(sbase)) : "memory", "m0");
}
// A pointer to device memory that came out of the kernel's argument words, as one the compiler knows to be
// global: it emits flat accesses otherwise, which hold up every wait for an LDS read too
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* as_global(T* p) {
    return (__attribute__((address_space(1))) T*)p;
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The group's header (everything before p[]) and one problem record are fetched as a few wide
// scalar loads (dword-aligned vector types)
typedef uint32_t u32x16u __attribute__((ext_vector_type(16), aligned(4)));
typedef uint32_t u32x8u __attribute__((ext_vector_type(8), aligned(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(4)));
struct alignas(8) ProblemWords { uint32_t w[48]; };
static_assert(offsetof(GemmGroup, p) == 88 && offsetof(GemmGroup, first_tile) == 24 && offsetof(GemmGroup, zero_ptr) == 16 &&
              offsetof(GemmGroup, n_lead) == 8 && offsetof(GemmGroup, zero_n) == 12, "header layout");
static_assert(sizeof(GemmProblem) == sizeof(ProblemWords), "problem record size");

// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  Give every XCD a
// contiguous range of tiles, and order tiles inside a problem in bands of 8 row-tiles
// (row-tile index fastest), so that the workgroups resident on one XCD share a small set
// of activation rows and weight rows.
// The tiles of signalling problems (down-projections that tiles of this same launch wait
// for) come first and are dealt round-robin: they are the first workgroups dispatched on
// every XCD, so all of them are running, or done, before any tile can wait for them.  A few tiles of
// longer K loops may follow in the same manner (launch_cfg).
// Kernel arguments arrive through scalar loads, and the compiler issues a load next to its first
// use: left alone, a workgroup pays six or seven such rounds one after the other before its
// first operand load.  One round is forced instead, 0.4 us: the header and the first problem's record
// (made opaque right away, so no load can sink below); a tile of a later problem takes a second.
// False: a workgroup beyond the last tile.
struct ProblemRegs { u32x16u a, b; u32x8u c; u32x4u d, e; };
__device__ __forceinline__ void load_problem(const GemmProblem& p, ProblemRegs& r) {
    const uint32_t* const pw = reinterpret_cast<const uint32_t*>(&p);
    r.a = *reinterpret_cast<const u32x16u*>(pw);
    r.b = *reinterpret_cast<const u32x16u*>(pw + 16);
    r.c = *reinterpret_cast<const u32x8u*>(pw + 32);
    r.d = *reinterpret_cast<const u32x4u*>(pw + 40);
    r.e = *reinterpret_cast<const u32x4u*>(pw + 44);
}
__device__ __forceinline__ bool gemm_pick_tile(const GemmGroup& g, int& tile, GemmProblem& P, int& zero_n, int32_t*& zero_ptr) {
    const uint32_t* const hw = reinterpret_cast<const uint32_t*>(&g);
    u32x16u ha = *reinterpret_cast<const u32x16u*>(hw);
    u32x4u hb = *reinterpret_cast<const u32x4u*>(hw + 16);
    u32x2u hc = *reinterpret_cast<const u32x2u*>(hw + 20);
    ProblemRegs r;
    load_problem(g.p[0], r);
    asm volatile("" : "+s"(ha), "+s"(hb), "+s"(hc), "+s"(r.a), "+s"(r.b), "+s"(r.c), "+s"(r.d), "+s"(r.e));
    const int total = (int)ha[1], lead = (int)ha[2], np = (int)ha[0];
    zero_n = (int)ha[3];
    zero_ptr = reinterpret_cast<int32_t*>(((uint64_t)ha[5] << 32) | ha[4]);
    tile = blockIdx.x;
    if (tile >= lead) {
        const int per = (total - lead + 7) >> 3, i = tile - lead;   // the grid holds a multiple of 8 beyond the leading tiles
        tile = lead + (i & 7) * per + (i >> 3);
        if (tile >= total) return false;
    }
    if (np > 1) {
        int pi = 0;
#pragma unroll
        for (int i = 1; i < GEMM_MAX_PROBLEMS; ++i) {
            const int ft = (int)(i < 10 ? ha[6 + i] : i < 14 ? hb[i - 10] : hc[i - 14]);
            if (i < np && tile >= ft) pi = i;
        }
        if (pi) {
            load_problem(g.p[pi], r);
            asm volatile("" : "+s"(r.a), "+s"(r.b), "+s"(r.c), "+s"(r.d), "+s"(r.e));
        }
    }
    ProblemWords words;
#pragma unroll
    for (int i = 0; i < 16; ++i) { words.w[i] = r.a[i]; words.w[16 + i] = r.b[i]; }
#pragma unroll
    for (int i = 0; i < 8; ++i) words.w[32 + i] = r.c[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) { words.w[40 + i] = r.d[i]; words.w[44 + i] = r.e[i]; }
    P = __builtin_bit_cast(GemmProblem, words);
    return true;
}

}  // namespace sd
