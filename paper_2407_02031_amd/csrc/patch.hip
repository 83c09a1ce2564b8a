// In-place LoRA patching for gfx950: W <- W + scale * (B A) over a list of fp32 matrices in
// one grouped launch, with W's old bits saved to an undo record in the same pass, and the
// inverse pass that copies them back (Section 4.2, "Efficient LoRA patching": merge into the
// base parameters in place; take the adapter off after the request).
//
// HBM-bound: 4 B read + 4 B write (+ 4 B undo) per element against 2r FLOP, so the rank-r
// product must not become the limit: it runs on the fp32 matrix cores (32x32x2 MFMA) while
// the W loads of the same tile are in flight.  One wavefront owns 32 rows x 128 columns;
// lane l holds columns c0 + 4*(l%32) + {0..3} of 16 rows, i.e. four MFMA column blocks
// interleaved so that every W access is a 16-byte float4 and a wavefront load covers two
// 512-byte row segments.
#include "common.hpp"

namespace sd {

// streaming accesses: W, W' and the undo record are touched exactly once per pass
typedef float nt_f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 nt_load4(const float* p) {
    nt_f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const nt_f32x4*>(p));
    return float4{t[0], t[1], t[2], t[3]};
}
__device__ __forceinline__ void nt_store4(float* p, float4 v) {
    nt_f32x4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<nt_f32x4*>(p));
}
#define NT_LOAD4(p) nt_load4(p)
#define NT_STORE4(p, v) nt_store4(p, v)

// These kernels stream: what limits them is how well HBM copes with the mix of requests in
// flight, and past a point more wavefronts per CU make that worse (more streams interleaved per
// channel).  The copies back therefore ask for dynamic LDS that no kernel touches, only to cap the
// workgroups (of two wavefronts) per CU (160 KB of LDS): eight for the plain copy (a sweep's 310 matrices 1.09 ms,
// 1.11 with ten or six), six where the bf16 copy is written too (1.43 ms; 1.54 with ten or with 16 wavefronts in
// workgroups of four).  The patch passes are held to 8 to 12 wavefronts per CU by registers and LDS.
constexpr int UNPATCH_THROTTLE_LDS = 20 * 1024, UNPATCH_MULTI_THROTTLE_LDS = 26 * 1024;

struct PatchPlanEntry {
    sd_patch_desc d;       // 48 bytes
    int64_t tile_begin;    // first tile of this matrix
    int32_t tiles_c;       // tiles side by side
    int32_t ntiles;        // tiles of this matrix
};
static_assert(sizeof(sd_patch_desc) == 48, "descriptor layout");
static_assert(sizeof(PatchPlanEntry) == 64, "plan entry layout");

struct PatchMultiEntry {
    sd_patch_multi_desc d;
    int64_t tile_begin;
    int32_t tiles_c;
    int32_t ntiles;
};
static_assert(sizeof(PatchMultiEntry) % 8 == 0, "plan entry layout");

// A plan counts tiles of PLAN_ROWS x PT_COLS.  A workgroup has two wavefronts of 32 rows x 128 columns side
// by side for each of the PT_WR tiles, one above the other, that it takes together.  With PT_WR = 2, matrix i
// has the workgroups from workgroups_before(i) on, half its tiles rounded up, and at most one before matrix
// i + 1 that finds nothing to do.
constexpr int PLAN_ROWS = 32, PT_WC = 2, PT_COLS = 128 * PT_WC;
constexpr int UNPATCH_THREADS = 128;
template <int PT_WR>
__host__ __device__ __forceinline__ int64_t workgroups_before(int64_t tile_begin, int i) { return PT_WR == 1 ? tile_begin : (tile_begin + i + 1) >> 1; }

// the matrix of workgroup wg and, in `local`, its number among that matrix's `count` workgroups
template <int PT_WR, typename Entry>
__device__ __forceinline__ int find_entry(const Entry* __restrict__ plan, int n, int64_t wg, int& local, int& count) {
    int lo = 0, hi = n - 1;   // last entry that begins at or before wg
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (workgroups_before<PT_WR>(plan[mid].tile_begin, mid) <= wg) lo = mid; else hi = mid - 1;
    }
    local = (int)(wg - workgroups_before<PT_WR>(plan[lo].tile_begin, lo));
    count = (plan[lo].ntiles + PT_WR - 1) / PT_WR;
    return lo;
}

// ---------------------------------------------------------------------------------------
// The product's operands come through LDS.  A wavefront that fetches its own A and B fragments
// from L2 pays a round trip per batch of them, on top of the matrix-core time that it issues in
// order; with ranks of 16 and 64 on one matrix those trips were two thirds of the pass.  Here the
// workgroup's A columns and B rows of PT_RC ranks at a time go straight from global memory into a
// ring of LDS stages, all but one of them requested right behind the W tile, shared by the
// workgroup's wavefronts, and refilled while the chunks in between multiply: no rank has a round
// trip between its first and its last MFMA.
//
// Measured, fragments from L2 and now: 310 matrices (830 M elements) under rank 32 1720 and 1718 us (1680 at
// the 6.0 TB/s that the copy back reaches), rank 64 2550 and 1967, two of rank 32 with the bf16 copy 2509 and 2040
// (1980); 60 matrices of 1280 x 1280 under ranks 16 and 64, on and off, 499 and 424.  Scalars are the scarce resource:
// bounds and row addresses are formed where they are used and not carried through the products or
// around the loop over a workgroup's possible second tile (spilled, they cost 6 to 10 %).
// ---------------------------------------------------------------------------------------
constexpr int PT_RC = 16;
constexpr int PT_A_CHUNKS = PT_RC * PT_COLS / 4;    // 16-byte chunks of a stage: A rows [rank][PT_COLS] ...
constexpr int PT_B_CHUNKS = PLAN_ROWS * PT_RC / 4;  // ... then, for each of the PT_WR tiles, B rows [row][PT_RC], chunks of a row XOR-swizzled
template <int PT_WR>
constexpr int PT_STAGE_CHUNKS = PT_A_CHUNKS + PT_WR * PT_B_CHUNKS;
static_assert(PT_RC == 16 && PT_COLS == 256 && PT_B_CHUNKS == 64 * PT_WC, "stage layout");

// where lanes point whose chunk lies past the rank or the matrix
__device__ __attribute__((aligned(256))) uint32_t g_patch_zeros[64];

// one direct global -> LDS load: each lane fetches 16 bytes, the 64 pieces land contiguously at LDS
// byte address lds_base (wave-uniform); completion is tracked with vmcnt and a barrier
__device__ __forceinline__ void patch_dma16(const void* gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(gptr) : "memory", "m0");
}
// ... each lane 4 bytes, 256 in all
__device__ __forceinline__ void patch_dma4(const void* gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(gptr) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void patch_wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// one matrix's adapters, in application order
struct PatchAdapters {
    const float* const* A;
    const float* const* B;
    const int32_t* r;
    const float* scale;
    int n;
};

// A workgroup tile under the adapters of its matrix: W_i = fl32(W_{i-1} + fl32(scale_i * (B_i A_i))),
// undo <- W_0, W <- W_n, serving <- bf16(W_n).  For in a multiple of 4 (a lane's four columns are inside
// the matrix or outside together) and any rank: a B whose rows are not 16-byte aligned comes in 4 bytes
// at a time (60 matrices of 1280 x 1280 under rank 33: %ODD%).  Wavefronts and
// lanes outside the matrix load and multiply with the others and store nothing.
// Lane l of a wavefront holds columns c0 + 4 * (l % 32) + {0..3} of 16 rows; with the 32x32x2 MFMA
// the upper half-wavefront supplies ranks 4 .. 7 of every 8, the lower half ranks 0 .. 3, so that one
// 16-byte LDS read holds a lane's B values of 8 ranks.
template <int PT_WR, int PT_STAGES>
__device__ __forceinline__ void patch_tile(float* __restrict__ W, float* __restrict__ Und, uint16_t* __restrict__ S, int out, int in,
                                           const PatchAdapters& ad, int tr, int tc, u32x4* const lds) {
    constexpr int NW = PT_WR * PT_WC, STAGE = PT_STAGE_CHUNKS<PT_WR>;
    // direct-to-LDS loads of a wavefront per stage: of A, and one of B or, where its rows are not 16-byte aligned, four
    constexpr int A_LOADS = PT_A_CHUNKS / 64 / NW, LOADS = A_LOADS + 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int row_wg = tr * (PLAN_ROWS * PT_WR), col_wg = tc * PT_COLS;
    const int r0 = row_wg + (wave / PT_WC) * 32, c0 = col_wg + (wave % PT_WC) * 128;
    const int col = c0 + 4 * l32;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds + wave * 1024;

    // ---- operand chunks: (adapter, first rank), walked by the loads a few ahead of the MFMAs
    int ia = 0, ik = 0;            // next chunk to request
    bool half = false;             // the chunk last requested had 8 ranks or fewer: half of A's loads
    int r = ad.r[0];
    const float* A = ad.A[0];
    const float* B = ad.B[0];
    auto issue = [&](int slot) {
        const uint32_t dst = lds_base + slot * (STAGE * 16);
        half = ik + 8 >= r;
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j) {       // one rank's 256 columns
            if (j == A_LOADS / 2 && half) break;
            const int k = ik + j * NW + wave, c = col_wg + lane * 4;
            patch_dma16(k < r && c < in ? (const void*)(A + (size_t)k * in + c) : (const void*)g_patch_zeros, dst + j * (NW * 1024));
        }
        const uint32_t bdst = dst + A_LOADS * (NW * 1024);
        if ((r & 3) == 0) {                          // this wavefront's 16 rows of B, 4 ranks per lane
            const int row = wave * 16 + (lane >> 2), k = ik + (((lane & 3) ^ ((row >> 2) & 3)) << 2);
            patch_dma16(k < r && row_wg + row < out ? (const void*)(B + (size_t)(row_wg + row) * r + k) : (const void*)g_patch_zeros, bdst);
        } else {                                     // ... one rank per lane, in the same places
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = wave * 16 + j * 4 + (lane >> 4), k = ik + ((((lane >> 2) & 3) ^ ((row >> 2) & 3)) << 2) + (lane & 3);
                patch_dma4(k < r && row_wg + row < out ? (const void*)(B + (size_t)(row_wg + row) * r + k) : (const void*)g_patch_zeros, bdst + j * 256);
            }
        }
        ik += PT_RC;
        if (ik >= r && ++ia < ad.n) {
            ik = 0;
            r = ad.r[ia];
            A = ad.A[ia];
            B = ad.B[ia];
        }
    };
    int total = 0;                 // chunks in all
    for (int a = 0; a < ad.n; ++a) total += (ad.r[a] + PT_RC - 1) / PT_RC;
    auto first_chunks = [&]() {    // all stages but one
#pragma unroll
        for (int s = 0; s < PT_STAGES - 1; ++s)
            if (s < total) issue(s);
    };

    // ---- W, undo and serving addresses: the row of register v lies 8 * (v / 4) + v % 4 rows below
    // the lane's first, a wave-uniform distance; one 32-bit byte offset per lane, from the wavefront's
    // first element, serves all arrays (the caller checked that in < 2^27)
    const size_t first = (size_t)r0 * in + c0;
    W += first;
    Und += first;
    if (S) S += first;
    const uint32_t woff = ((uint32_t)(4 * hi) * (uint32_t)in + 4 * l32) * 4;
    auto row_of = [&](int v) { return 8 * (v >> 2) + (v & 3); };
    auto row_bytes = [&](int v) -> size_t { return (size_t)row_of(v) * in * 4; };
    const bool full = r0 + 32 <= out && c0 + 128 <= in;     // uniform: no lane of this wavefront is outside
    const bool col_in = col < in;
    float4 w[16];
    if (full) {
#pragma unroll
        for (int v = 0; v < 16; ++v) w[v] = NT_LOAD4(reinterpret_cast<const float*>(reinterpret_cast<const char*>(W) + row_bytes(v) + woff));
        first_chunks();
        // W's old bits go out first, as one burst of stores, before any adapter's product
#pragma unroll
        for (int v = 0; v < 16; ++v) NT_STORE4(reinterpret_cast<float*>(reinterpret_cast<char*>(Und) + row_bytes(v) + woff), w[v]);
        patch_wait_vmcnt<16>();    // the chunks have landed, the stores may be on their way
    } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            w[v] = float4{0.f, 0.f, 0.f, 0.f};
            if (col_in && r0 + 4 * hi + row_of(v) < out) w[v] = NT_LOAD4(reinterpret_cast<const float*>(reinterpret_cast<const char*>(W) + row_bytes(v) + woff));
        }
        first_chunks();
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (col_in && r0 + 4 * hi + row_of(v) < out) NT_STORE4(reinterpret_cast<float*>(reinterpret_cast<char*>(Und) + row_bytes(v) + woff), w[v]);
        patch_wait_vmcnt<0>();
    }

    f32x16 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    int ma = 0, mk = 0, slot = 0;  // adapter and first rank of the chunk being multiplied, its ring slot
    int mr = ad.r[0];
    float scale = ad.scale[0];
    const int brow = (wave / PT_WC) * 32 + l32;
#pragma unroll 1
    for (int c = 0; c < total; ++c) {
        static_assert(PT_STAGES == 2 || PT_STAGES == 3, "at most one chunk is in flight behind the one waited for");
        if (c >= PT_STAGES - 1) {  // (a chunk behind it with more loads than LOADS: some of those are waited for too)
            if (PT_STAGES == 3 && c + 1 < total && !half) patch_wait_vmcnt<LOADS>();
            else if (PT_STAGES == 3 && c + 1 < total) patch_wait_vmcnt<A_LOADS / 2 + 1>();
            else patch_wait_vmcnt<0>();
        }
        __syncthreads();           // every wavefront's part of the chunk is in LDS, and the slot before it is free
        if (c + PT_STAGES - 1 < total) issue(slot == 0 ? PT_STAGES - 1 : slot - 1);
        const u32x4* const la = lds + slot * STAGE;
        const u32x4* const lb = la + PT_A_CHUNKS;
#pragma unroll
        for (int u = 0; u < PT_RC / 8; ++u) {
            if (u > 0 && mk + 8 * u >= mr) break;      // nothing but zeros: a rank of 8 has half the matrix-core time
            const float4 bv = __builtin_bit_cast(float4, lb[brow * 4 + ((2 * u + hi) ^ ((brow >> 2) & 3))]);
            float4 av[4];
#pragma unroll
            for (int kp = 0; kp < 4; ++kp) av[kp] = __builtin_bit_cast(float4, la[(8 * u + 4 * hi + kp) * (PT_COLS / 4) + (wave % PT_WC) * 32 + l32]);
#pragma unroll
            for (int kp = 0; kp < 4; ++kp) {
                const float b = reinterpret_cast<const float*>(&bv)[kp];
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(b, av[kp].x, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(b, av[kp].y, acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(b, av[kp].z, acc[2], 0, 0, 0);
                acc[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(b, av[kp].w, acc[3], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        slot = slot + 1 == PT_STAGES ? 0 : slot + 1;
        mk += PT_RC;
        if (mk >= mr) {            // the adapter's last chunk
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                w[v].x = __fadd_rn(w[v].x, __fmul_rn(scale, acc[0][v]));
                w[v].y = __fadd_rn(w[v].y, __fmul_rn(scale, acc[1][v]));
                w[v].z = __fadd_rn(w[v].z, __fmul_rn(scale, acc[2][v]));
                w[v].w = __fadd_rn(w[v].w, __fmul_rn(scale, acc[3][v]));
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
            mk = 0;
            if (++ma < ad.n) {
                mr = ad.r[ma];
                scale = ad.scale[ma];
            }
        }
    }
    // (the offset and the lane's row are laundered so that row addresses and bounds are formed again here
    // instead of being carried, or spilled, through the adapters' products)
    uint32_t woff2 = woff;
    int row2 = r0 + 4 * hi;
    asm volatile("" : "+v"(woff2), "+v"(row2));
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        if (full || (col_in && row2 + row_of(v) < out)) {
            NT_STORE4(reinterpret_cast<float*>(reinterpret_cast<char*>(W) + row_bytes(v) + woff2), w[v]);
            if (S) {
                bf16x4 o = {(__bf16)w[v].x, (__bf16)w[v].y, (__bf16)w[v].z, (__bf16)w[v].w};
                *reinterpret_cast<bf16x4*>(reinterpret_cast<char*>(S) + row_bytes(v) / 2 + woff2 / 2) = o;
            }
        }
    }
}

// The same for rows that are not 16-byte aligned (in no multiple of 4): every access guarded, one
// element at a time.  Lane l holds columns l % 32 of the four 32-column blocks, so that a half-wavefront
// still touches 128 contiguous bytes (%RAG%).
template <int PT_WR>
__device__ __forceinline__ void patch_tile_any(float* __restrict__ W, float* __restrict__ Und, uint16_t* __restrict__ S, int out, int in,
                                               const PatchAdapters& ad, int tr, int tc) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, hi = lane >> 5;
    const int r0 = tr * (PLAN_ROWS * PT_WR) + (wave / PT_WC) * 32;
    const int col = tc * PT_COLS + (wave % PT_WC) * 128 + l32;
    float w[16][4];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int row = min(r0 + 8 * (v >> 2) + 4 * hi + (v & 3), out - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) w[v][j] = W[(size_t)row * in + min(col + 32 * j, in - 1)];   // (outside: an element that is inside, not stored)
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int row = r0 + 8 * (v >> 2) + 4 * hi + (v & 3);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (row < out && col + 32 * j < in) Und[(size_t)row * in + col + 32 * j] = w[v][j];
    }
    const int brow = r0 + l32;
#pragma unroll 1
    for (int a = 0; a < ad.n; ++a) {
        f32x16 acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
        const float* const A = ad.A[a];
        const float* const B = ad.B[a];
        const int r = ad.r[a];
#pragma unroll 1
        for (int kp = 0; kp < 4 * ((r + 7) >> 3); ++kp) {
            const int kk = (kp >> 2) * 8 + 4 * hi + (kp & 3);   // same pairs of ranks as above: same bits
            const bool kv = kk < r;
            const float bv = (kv && brow < out) ? B[(size_t)brow * r + kk] : 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float av = (kv && col + 32 * j < in) ? A[(size_t)kk * in + col + 32 * j] : 0.f;
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv, av, acc[j], 0, 0, 0);
            }
        }
        const float scale = ad.scale[a];
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) w[v][j] = __fadd_rn(w[v][j], __fmul_rn(scale, acc[j][v]));
    }
    int row2 = r0 + 4 * hi, col2 = col;     // laundered, as above
    asm volatile("" : "+v"(row2), "+v"(col2));
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int row = row2 + 8 * (v >> 2) + (v & 3);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (row >= out || col2 + 32 * j >= in) continue;
            const size_t idx = (size_t)row * in + col2 + 32 * j;
            W[idx] = w[v][j];
            if (S) S[idx] = __builtin_bit_cast(uint16_t, (__bf16)w[v][j]);
        }
    }
}

template <int PT_WR, int PT_STAGES>
__device__ __forceinline__ void patch_matrix_tile(float* W, float* Und, uint16_t* S, int out, int in, const PatchAdapters& ad, int local, int tiles_c,
                                                  u32x4* const lds) {
    const bool quads = (in & 3) == 0 && in < (1 << 27);
    // pairs of the plan's tiles, then, under an odd number of tile rows, the last row two side by side
    int tr = local / tiles_c, tc = local % tiles_c, end = tc + 1;
    if (PT_WR == 2) {
        const int tile_rows = (out + PLAN_ROWS - 1) / PLAN_ROWS, pairs = tiles_c * (tile_rows >> 1);
        if (local >= pairs) {
            tr = tile_rows >> 1;
            tc = 2 * (local - pairs);
            end = min(tc + 2, tiles_c);
        }
    }
#pragma unroll 1
    for (; tc < end; ++tc) {
        asm volatile("" : "+s"(tr), "+s"(out), "+s"(in));     // (nothing of a tile is carried, or spilled, around the loop)
        if (quads) patch_tile<PT_WR, PT_STAGES>(W, Und, S, out, in, ad, tr, tc, lds);
        else patch_tile_any<PT_WR>(W, Und, S, out, in, ad, tr, tc);
        if (PT_WR == 1) break;
        if (tc + 1 < end) __syncthreads();      // the next tile's loads reuse the ring
    }
}

template <int PT_WR, int STAGES>
__global__ __launch_bounds__(128 * PT_WR, 2) void lora_patch_kernel(const PatchPlanEntry* __restrict__ plan, int n) {
    __shared__ u32x4 lds[STAGES * PT_STAGE_CHUNKS<PT_WR>];
    int local, count;
    const PatchPlanEntry& E = plan[find_entry<PT_WR>(plan, n, blockIdx.x, local, count)];
    if (local >= count) return;
    const PatchAdapters ad = {&E.d.A, &E.d.B, &E.d.r, &E.d.scale, 1};
    patch_matrix_tile<PT_WR, STAGES>(E.d.W, E.d.undo, nullptr, E.d.out, E.d.in, ad, local, E.tiles_c, lds);
}

// Several adapters on one matrix in one pass over W (one or two LoRAs per request is the norm,
// Section 3.1; each is merged as in Section 4.2): the tile's W values stay in registers while
// the adapters are applied one after the other, so the result equals successive single patches bit
// for bit at one third of their traffic for two adapters.  Optionally also writes the bf16 copy of
// W' that the bf16 GEMMs read.
template <int PT_WR, int STAGES>
__global__ __launch_bounds__(128 * PT_WR, PT_WR + 1) void lora_patch_multi_kernel(const PatchMultiEntry* __restrict__ plan, int n) {
    __shared__ u32x4 lds[STAGES * PT_STAGE_CHUNKS<PT_WR>];
    int local, count;
    const PatchMultiEntry& E = plan[find_entry<PT_WR>(plan, n, blockIdx.x, local, count)];
    if (local >= count) return;
    const PatchAdapters ad = {E.d.A, E.d.B, E.d.r, E.d.scale, E.d.n_adapters};
    patch_matrix_tile<PT_WR, STAGES>(E.d.W, E.d.undo, E.d.serving, E.d.out, E.d.in, ad, local, E.tiles_c, lds);
}

// W <- undo (flat linear copy), and the serving copy follows it: bf16(undo)
__global__ __launch_bounds__(UNPATCH_THREADS) void lora_unpatch_multi_kernel(const PatchMultiEntry* __restrict__ plan, int n) {
    int local, count;
    const PatchMultiEntry& E = plan[find_entry<1>(plan, n, blockIdx.x, local, count)];
    float* __restrict__ W = E.d.W;
    const float* __restrict__ U = E.d.undo;
    uint16_t* __restrict__ S = E.d.serving;
    const int64_t elems = (int64_t)E.d.out * E.d.in;
    // the matrix's workgroups sweep it together, see lora_unpatch_kernel
    const int64_t stride = (int64_t)count * UNPATCH_THREADS * 4;
    int64_t i = ((int64_t)local * UNPATCH_THREADS + threadIdx.x) * 4;
#pragma unroll 4
    for (; i + 4 <= elems; i += stride) {
        const float4 v = NT_LOAD4(U + i);
        NT_STORE4(W + i, v);
        if (S) {
            bf16x4 o = {(__bf16)v.x, (__bf16)v.y, (__bf16)v.z, (__bf16)v.w};
            *reinterpret_cast<bf16x4*>(S + i) = o;
        }
    }
    if (i < elems)   // the matrix's last 1..3 elements
        for (int64_t j = i; j < elems; ++j) {
            W[j] = U[j];
            if (S) S[j] = __builtin_bit_cast(uint16_t, (__bf16)U[j]);
        }
}

// Unpatch: W <- undo, a pure copy.  The matrix's workgroups (as many as the patch pass used)
// sweep it together as one flat array: in every round workgroup w copies the w-th 2 KB, so all
// that is in flight at any moment is one narrow, contiguous window of the matrix.  HBM likes
// that best: 6.0 TB/s, against 5.6 when every workgroup copies a contiguous 32 KB of its own.
__global__ __launch_bounds__(UNPATCH_THREADS) void lora_unpatch_kernel(const PatchPlanEntry* __restrict__ plan, int n) {
    int local, count;
    const PatchPlanEntry& E = plan[find_entry<1>(plan, n, blockIdx.x, local, count)];
    float* __restrict__ W = E.d.W;
    const float* __restrict__ U = E.d.undo;
    const int64_t elems = (int64_t)E.d.out * E.d.in;
    const int64_t stride = (int64_t)count * UNPATCH_THREADS * 4;
    int64_t i = ((int64_t)local * UNPATCH_THREADS + threadIdx.x) * 4;
#pragma unroll 4
    for (; i + 4 <= elems; i += stride) NT_STORE4(W + i, NT_LOAD4(U + i));
    if (i < elems)   // the matrix's last 1..3 elements
        for (int64_t j = i; j < elems; ++j) W[j] = U[j];
}

}  // namespace sd

using namespace sd;

extern "C" size_t sd_patch_plan_bytes(int32_t n) { return n > 0 ? (size_t)n * sizeof(PatchPlanEntry) : 0; }

extern "C" int sd_patch_plan_build(const sd_patch_desc* descs, int32_t n, void* plan_host, size_t plan_bytes,
                                   int64_t* total_tiles) {
    SD_REQUIRE(n >= 0, SD_EINVAL, "patch plan: n=%d", n);
    SD_REQUIRE(total_tiles, SD_EINVAL, "patch plan: total_tiles is null");
    *total_tiles = 0;
    if (n == 0) return SD_OK;
    SD_REQUIRE(descs && plan_host, SD_EINVAL, "patch plan: null pointer");
    SD_REQUIRE(plan_bytes >= sd_patch_plan_bytes(n), SD_EWORKSPACE, "patch plan: buffer of %zu bytes, need %zu", plan_bytes,
               sd_patch_plan_bytes(n));
    PatchPlanEntry* plan = static_cast<PatchPlanEntry*>(plan_host);
    int64_t total = 0;
    for (int i = 0; i < n; ++i) {
        const sd_patch_desc& d = descs[i];
        SD_REQUIRE(d.W && d.A && d.B && d.undo, SD_EINVAL, "patch desc %d: null pointer (W, A, B and undo are required)", i);
        SD_REQUIRE(aligned16(d.W) && aligned16(d.A) && aligned16(d.B) && aligned16(d.undo), SD_EINVAL,
                   "patch desc %d: pointers must be 16-byte aligned", i);
        SD_REQUIRE(d.out > 0 && d.in > 0 && d.r > 0 && d.r <= 1024, SD_EINVAL, "patch desc %d: out=%d in=%d r=%d", i, d.out, d.in, d.r);
        SD_REQUIRE(d.undo != d.W, SD_EINVAL, "patch desc %d: undo aliases W", i);
        plan[i].d = d;
        plan[i].tile_begin = total;
        plan[i].tiles_c = (d.in + PT_COLS - 1) / PT_COLS;
        const int64_t nt = (int64_t)plan[i].tiles_c * ((d.out + PLAN_ROWS - 1) / PLAN_ROWS);
        SD_REQUIRE(nt < (int64_t)0x7fffffff, SD_EUNSUPPORTED, "patch desc %d: too many tiles", i);
        plan[i].ntiles = (int32_t)nt;
        total += nt;
    }
    SD_REQUIRE(total < (int64_t)0x7fffffff, SD_EUNSUPPORTED, "patch plan: %lld tiles exceed one grid", (long long)total);
    *total_tiles = total;
    return SD_OK;
}

// Which workgroups a pass gets.  Up to two tiles per CU: one tile each, two workgroups with a three-stage ring on a
// CU (1 x 1280 x 1280 under rank 32 8.4 us, 9.5 in pairs of tiles; under 8 and 8 8.0 and 9.3).  Up to three: one tile
// each with two stages, which fit four times (3 x 1280 x 1280 under rank 8 12.4, 14.7 in pairs, which leave some CUs two
// and most one; 14.4 with three stages).  Beyond that pairs, which share A's stages: 4 x 1280 x 1280 under 8 and 8 17.6, 19.3
// and 21.2; 60 under 16 and 64 271, 297 and 370.  One adapter: three stages and two workgroups per CU; several: two stages,
// which leaves room for a third workgroup.
constexpr int64_t SINGLE_3_STAGES = 2 * 256, SINGLE_2_STAGES = 3 * 256;
static int patch_launch(bool undo, const void* plan_dev, int32_t n, int64_t total_tiles, void* stream) {
    SD_REQUIRE(n >= 0 && total_tiles >= 0, SD_EINVAL, "patch: n=%d tiles=%lld", n, (long long)total_tiles);
    if (n == 0 || total_tiles == 0) return SD_OK;
    SD_REQUIRE(plan_dev, SD_EINVAL, "patch: plan is null");
    SD_REQUIRE(total_tiles < (int64_t)0x7fffffff, SD_EUNSUPPORTED, "patch: %lld tiles exceed one grid", (long long)total_tiles);
    const PatchPlanEntry* plan = static_cast<const PatchPlanEntry*>(plan_dev);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (SD_DRY_RUN(undo ? "unpatch; " : total_tiles <= SINGLE_3_STAGES ? "patch 1 tile/3 stages; " : total_tiles <= SINGLE_2_STAGES ? "patch 1 tile/2 stages; " : "patch 2 tiles/3 stages; "))
        return SD_OK;
    if (undo) hipLaunchKernelGGL(lora_unpatch_kernel, dim3((unsigned)total_tiles), dim3(UNPATCH_THREADS), UNPATCH_THROTTLE_LDS, s, plan, n);
    else if (total_tiles <= SINGLE_3_STAGES) hipLaunchKernelGGL((lora_patch_kernel<1, 3>), dim3((unsigned)total_tiles), dim3(128), 0, s, plan, n);
    else if (total_tiles <= SINGLE_2_STAGES) hipLaunchKernelGGL((lora_patch_kernel<1, 2>), dim3((unsigned)total_tiles), dim3(128), 0, s, plan, n);
    else hipLaunchKernelGGL((lora_patch_kernel<2, 3>), dim3((unsigned)((total_tiles + n + 1) >> 1)), dim3(256), 0, s, plan, n);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

extern "C" int sd_lora_patch(const void* plan_dev, int32_t n, int64_t total_tiles, void* stream) {
    return patch_launch(false, plan_dev, n, total_tiles, stream);
}
extern "C" int sd_lora_unpatch(const void* plan_dev, int32_t n, int64_t total_tiles, void* stream) {
    return patch_launch(true, plan_dev, n, total_tiles, stream);
}

extern "C" size_t sd_patch_multi_plan_bytes(int32_t n) { return n > 0 ? (size_t)n * sizeof(PatchMultiEntry) : 0; }

extern "C" int sd_patch_multi_plan_build(const sd_patch_multi_desc* descs, int32_t n, void* plan_host, size_t plan_bytes,
                                         int64_t* total_tiles) {
    SD_REQUIRE(n >= 0, SD_EINVAL, "patch plan: n=%d", n);
    SD_REQUIRE(total_tiles, SD_EINVAL, "patch plan: total_tiles is null");
    *total_tiles = 0;
    if (n == 0) return SD_OK;
    SD_REQUIRE(descs && plan_host, SD_EINVAL, "patch plan: null pointer");
    SD_REQUIRE(plan_bytes >= sd_patch_multi_plan_bytes(n), SD_EWORKSPACE, "patch plan: buffer of %zu bytes, need %zu", plan_bytes,
               sd_patch_multi_plan_bytes(n));
    PatchMultiEntry* plan = static_cast<PatchMultiEntry*>(plan_host);
    int64_t total = 0;
    for (int i = 0; i < n; ++i) {
        const sd_patch_multi_desc& d = descs[i];
        SD_REQUIRE(d.W && d.undo && aligned16(d.W) && aligned16(d.undo), SD_EINVAL, "patch desc %d: W and undo must be non-null and 16-byte aligned", i);
        SD_REQUIRE(d.undo != d.W, SD_EINVAL, "patch desc %d: undo aliases W", i);
        SD_REQUIRE(!d.serving || (reinterpret_cast<uintptr_t>(d.serving) & 7) == 0, SD_EINVAL, "patch desc %d: serving copy must be 8-byte aligned", i);
        SD_REQUIRE(d.out > 0 && d.in > 0, SD_EINVAL, "patch desc %d: out=%d in=%d", i, d.out, d.in);
        SD_REQUIRE(d.n_adapters >= 1 && d.n_adapters <= SD_PATCH_MAX_ADAPTERS, SD_EINVAL, "patch desc %d: %d adapters (1..%d)", i, d.n_adapters,
                   SD_PATCH_MAX_ADAPTERS);
        for (int a = 0; a < d.n_adapters; ++a) {
            SD_REQUIRE(d.A[a] && d.B[a] && aligned16(d.A[a]) && aligned16(d.B[a]), SD_EINVAL,
                       "patch desc %d adapter %d: A and B must be non-null and 16-byte aligned", i, a);
            SD_REQUIRE(d.r[a] > 0 && d.r[a] <= 1024, SD_EINVAL, "patch desc %d adapter %d: r=%d", i, a, d.r[a]);
        }
        plan[i].d = d;
        plan[i].tile_begin = total;
        plan[i].tiles_c = (d.in + PT_COLS - 1) / PT_COLS;
        const int64_t nt = (int64_t)plan[i].tiles_c * ((d.out + PLAN_ROWS - 1) / PLAN_ROWS);
        SD_REQUIRE(nt < (int64_t)0x7fffffff, SD_EUNSUPPORTED, "patch desc %d: too many tiles", i);
        plan[i].ntiles = (int32_t)nt;
        total += nt;
    }
    SD_REQUIRE(total < (int64_t)0x7fffffff, SD_EUNSUPPORTED, "patch plan: %lld tiles exceed one grid", (long long)total);
    *total_tiles = total;
    return SD_OK;
}

static int patch_multi_launch(bool undo, const void* plan_dev, int32_t n, int64_t total_tiles, void* stream) {
    SD_REQUIRE(n >= 0 && total_tiles >= 0, SD_EINVAL, "patch: n=%d tiles=%lld", n, (long long)total_tiles);
    if (n == 0 || total_tiles == 0) return SD_OK;
    SD_REQUIRE(plan_dev, SD_EINVAL, "patch: plan is null");
    SD_REQUIRE(total_tiles < (int64_t)0x7fffffff, SD_EUNSUPPORTED, "patch: %lld tiles exceed one grid", (long long)total_tiles);
    const PatchMultiEntry* plan = static_cast<const PatchMultiEntry*>(plan_dev);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (SD_DRY_RUN(undo ? "unpatch multi; " : total_tiles <= SINGLE_3_STAGES ? "patch multi 1 tile/3 stages; " : total_tiles <= SINGLE_2_STAGES ? "patch multi 1 tile/2 stages; " : "patch multi 2 tiles/2 stages; "))
        return SD_OK;
    if (undo) hipLaunchKernelGGL(lora_unpatch_multi_kernel, dim3((unsigned)total_tiles), dim3(UNPATCH_THREADS), UNPATCH_MULTI_THROTTLE_LDS, s, plan, n);
    else if (total_tiles <= SINGLE_3_STAGES) hipLaunchKernelGGL((lora_patch_multi_kernel<1, 3>), dim3((unsigned)total_tiles), dim3(128), 0, s, plan, n);
    else if (total_tiles <= SINGLE_2_STAGES) hipLaunchKernelGGL((lora_patch_multi_kernel<1, 2>), dim3((unsigned)total_tiles), dim3(128), 0, s, plan, n);
    else hipLaunchKernelGGL((lora_patch_multi_kernel<2, 2>), dim3((unsigned)((total_tiles + n + 1) >> 1)), dim3(256), 0, s, plan, n);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

extern "C" int sd_lora_patch_multi(const void* plan_dev, int32_t n, int64_t total_tiles, void* stream) {
    return patch_multi_launch(false, plan_dev, n, total_tiles, stream);
}
extern "C" int sd_lora_unpatch_multi(const void* plan_dev, int32_t n, int64_t total_tiles, void* stream) {
    return patch_multi_launch(true, plan_dev, n, total_tiles, stream);
}
