// LayerNorm (per token) and token-major GroupNorm(32) for gfx950, plus the dtype
// converters at the stack boundary.  All statistics in fp32, biased variance, two passes
// over register-resident (LayerNorm) or shift-centred (GroupNorm) data.  HBM-bound.
#include "common.hpp"
#include "read_ahead.hpp"

#include <algorithm>

namespace sd {

// ---------------------------------------------------------------------------------------
// LayerNorm: one wavefront per row, the row lives in registers (C <= 2048, C % 4 == 0).
// ---------------------------------------------------------------------------------------
constexpr int LN_MAXJ = 8;   // float4 chunks per lane: 64 lanes * 4 * 8 = 2048 channels

// JN: chunks per lane the row needs (C <= 256 * JN); R: rows per wavefront, all of whose loads
// are issued before the first is used (the kernel is a stream: bytes in flight are what counts).
// zero_ptr/zero_n: flags that a later launch of the same call expects to find cleared.
template <bool XF32, int JN, int R, bool AHEAD>
__global__ __launch_bounds__(256) void layernorm_kernel(const void* __restrict__ xv, const uint16_t* __restrict__ gamma,
                                                        const uint16_t* __restrict__ beta, float eps,
                                                        uint16_t* __restrict__ y, int M, int C, int32_t* zero_ptr, int zero_n, const std::conditional_t<AHEAD, ReadRanges, NoRanges> ra) {
    if constexpr (AHEAD) {
        const int wgs = (M + 4 * R - 1) / (4 * R);
        if ((int)blockIdx.x >= wgs) {
            read_ahead<8>(ra, (int)blockIdx.x - wgs, (int)threadIdx.x);
            return;
        }
    }
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < zero_n; i += 256) zero_ptr[i] = 0;
    const int lane = threadIdx.x & 63;
    const int row0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * R;
    if (row0 >= M) return;
    const int nch = C >> 2;   // 4-element chunks per row
    float v[R][JN][4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int row = min(row0 + r, M - 1);   // rows past the end repeat the last one and are not stored
#pragma unroll
        for (int j = 0; j < JN; ++j) {
            const int ch = lane + j * 64;
            if (ch < nch) {
                if (XF32) {
                    const float4 t = reinterpret_cast<const float4*>(static_cast<const float*>(xv) + (size_t)row * C)[ch];
                    v[r][j][0] = t.x; v[r][j][1] = t.y; v[r][j][2] = t.z; v[r][j][3] = t.w;
                } else {
                    const uint2 t = reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(xv) + (size_t)row * C)[ch];
                    v[r][j][0] = bf16lo_to_f32(t.x); v[r][j][1] = bf16hi_to_f32(t.x);
                    v[r][j][2] = bf16lo_to_f32(t.y); v[r][j][3] = bf16hi_to_f32(t.y);
                }
            } else {
                v[r][j][0] = v[r][j][1] = v[r][j][2] = v[r][j][3] = 0.f;
            }
        }
    }
    uint2 gg[JN], bb[JN];
#pragma unroll
    for (int j = 0; j < JN; ++j) {
        const int ch = lane + j * 64;
        gg[j] = ch < nch ? reinterpret_cast<const uint2*>(gamma)[ch] : make_uint2(0, 0);
        bb[j] = ch < nch ? reinterpret_cast<const uint2*>(beta)[ch] : make_uint2(0, 0);
    }
    const float inv_c = 1.0f / (float)C;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        // One pass over the registers for both moments, taken about the row's first element (a
        // sample of the row, so the variance below loses no digits to a large common offset),
        // and one reduction for the pair.
        const float shift = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v[r][0][0])));
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int j = 0; j < JN; ++j) {
            const int ch = lane + j * 64;
            if (ch < nch) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[r][j][e] -= shift;
                    s1 += v[r][j][e];
                    s2 += v[r][j][e] * v[r][j][e];
                }
            }
        }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        const float dmean = s1 * inv_c;                      // mean - shift
        const float var = fmaxf(s2 * inv_c - dmean * dmean, 0.f);
        const float rstd = rsqrtf(var + eps);
        if (row0 + r < M) {
#pragma unroll
            for (int j = 0; j < JN; ++j) {
                const int ch = lane + j * 64;
                if (ch < nch) {
                    const float o0 = (v[r][j][0] - dmean) * rstd * bf16lo_to_f32(gg[j].x) + bf16lo_to_f32(bb[j].x);
                    const float o1 = (v[r][j][1] - dmean) * rstd * bf16hi_to_f32(gg[j].x) + bf16hi_to_f32(bb[j].x);
                    const float o2 = (v[r][j][2] - dmean) * rstd * bf16lo_to_f32(gg[j].y) + bf16lo_to_f32(bb[j].y);
                    const float o3 = (v[r][j][3] - dmean) * rstd * bf16hi_to_f32(gg[j].y) + bf16hi_to_f32(bb[j].y);
                    uint2 o;
                    o.x = pack_bf16x2(o0, o1);
                    o.y = pack_bf16x2(o2, o3);
                    reinterpret_cast<uint2*>(y + (size_t)(row0 + r) * C)[ch] = o;
                }
            }
        }
    }
}

// rows per wavefront: whole-step timings favour one (more, smaller workgroups) over two or four
constexpr int LN_ROWS = 1;
template <bool XF32, int JN, int R>
static void launch_ln(const void* x, const uint16_t* gamma, const uint16_t* beta, float eps, uint16_t* y, int M, int C,
                      int32_t* zero_ptr, int zero_n, hipStream_t stream, const ReadRanges& ra) {
    const dim3 grid((M + 4 * R - 1) / (4 * R) + ra.wgs);
    if (ra.wgs) hipLaunchKernelGGL((layernorm_kernel<XF32, JN, R, true>), grid, dim3(256), 0, stream, x, gamma, beta, eps, y, M, C, zero_ptr, zero_n, ra);
    else hipLaunchKernelGGL((layernorm_kernel<XF32, JN, R, false>), grid, dim3(256), 0, stream, x, gamma, beta, eps, y, M, C, zero_ptr, zero_n, NoRanges{});
}

int launch_layernorm(const void* x, int x_f32, const uint16_t* gamma, const uint16_t* beta, float eps,
                     uint16_t* y, int M, int C, hipStream_t stream, int32_t* zero_ptr, int zero_n, ReadAhead* ahead) {
    SD_REQUIRE(C % 4 == 0 && C > 0 && C <= 64 * 4 * LN_MAXJ, SD_EUNSUPPORTED, "layernorm: C=%d (need C %% 4 == 0, C <= %d)", C,
               64 * 4 * LN_MAXJ);
    if (M <= 0) return zero_n > 0 ? launch_clear_flags(zero_ptr, zero_n, stream) : SD_OK;
    // read-ahead: 8 MB, in workgroups small enough to leave eight on a CU (4 MB: the queue falls behind; 12: the launch takes longer than they save)
    const ReadRanges ra = ahead ? ahead->take(8ull << 20, 512, 8) : ReadRanges{};
    if (SD_DRY_RUN("layernorm%s%s; ", zero_n > 0 ? " clear" : "", dry_ranges(ra))) return SD_OK;
    if (C <= 768) {          // SDXL's 320 and 640 channels: three chunks per lane
        if (x_f32) launch_ln<true, 3, LN_ROWS>(x, gamma, beta, eps, y, M, C, zero_ptr, zero_n, stream, ra);
        else launch_ln<false, 3, LN_ROWS>(x, gamma, beta, eps, y, M, C, zero_ptr, zero_n, stream, ra);
    } else if (C <= 1280) {
        if (x_f32) launch_ln<true, 5, 1>(x, gamma, beta, eps, y, M, C, zero_ptr, zero_n, stream, ra);
        else launch_ln<false, 5, 1>(x, gamma, beta, eps, y, M, C, zero_ptr, zero_n, stream, ra);
    } else {
        if (x_f32) launch_ln<true, LN_MAXJ, 1>(x, gamma, beta, eps, y, M, C, zero_ptr, zero_n, stream, ra);
        else launch_ln<false, LN_MAXJ, 1>(x, gamma, beta, eps, y, M, C, zero_ptr, zero_n, stream, ra);
    }
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

// ---------------------------------------------------------------------------------------
// dtype converters (n % 4 == 0 handled by the tail loop)
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void cvt_bf16_f32_kernel(const uint16_t* __restrict__ x, float* __restrict__ y, size_t n) {
    size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i + 3 < n) {
        const uint2 t = *reinterpret_cast<const uint2*>(x + i);
        float4 o = {bf16lo_to_f32(t.x), bf16hi_to_f32(t.x), bf16lo_to_f32(t.y), bf16hi_to_f32(t.y)};
        *reinterpret_cast<float4*>(y + i) = o;
    } else {
        for (; i < n; ++i) y[i] = bf16_to_f32(x[i]);
    }
}
__global__ __launch_bounds__(256) void cvt_f32_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, size_t n) {
    size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i + 3 < n) {
        const float4 t = *reinterpret_cast<const float4*>(x + i);
        uint2 o;
        o.x = pack_bf16x2(t.x, t.y);
        o.y = pack_bf16x2(t.z, t.w);
        *reinterpret_cast<uint2*>(y + i) = o;
    } else {
        for (; i < n; ++i) y[i] = (uint16_t)f32_to_bf16_bits(x[i]);
    }
}
int launch_cvt_bf16_to_f32(const uint16_t* x, float* y, size_t n, hipStream_t stream) {
    if (!n || SD_DRY_RUN("convert; ")) return SD_OK;
    hipLaunchKernelGGL(cvt_bf16_f32_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, stream, x, y, n);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}
int launch_cvt_f32_to_bf16(const float* x, uint16_t* y, size_t n, hipStream_t stream) {
    if (!n || SD_DRY_RUN("convert; ")) return SD_OK;
    hipLaunchKernelGGL(cvt_f32_bf16_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, stream, x, y, n);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

// ---------------------------------------------------------------------------------------
// GroupNorm, token-major [Bn, T, C].  Pass 1: per (sample, chunk of tokens, group) sums of
// (x - shift) and (x - shift)^2 with shift = the group's first element in the sample
// (shifted-data variance: no catastrophic cancellation for data with a large mean).
// Pass 2: every workgroup combines the chunk partials of its sample in a fixed order (there is no
// finalize launch in between) and normalises its tokens.
//
// HBM-bound: x is read twice (the second time mostly out of the last-level cache) and y written
// once.  Both passes are streams, so a thread moves 16 bytes (VEC = 8 channels) per access and has
// all of its accesses in flight at once: a workgroup is `rows` tokens x C / VEC threads wide and
// takes up to GN_ITERS of such slabs.  Combining the partials is the other cost, nchunks * groups pairs
// per workgroup, and for short samples the chain of it is the pass: so a partial workgroup takes
// GN_PSLABS slabs at least, a thread fetches GN_RUN partials at once, and the sums in LDS are unrolled.
// us with SiLU, 4-byte accesses and 8-token workgroups / one slab per partial workgroup of 1024 threads
// and partials fetched one after the other / this way: 2 x 16384 x 320 42.7 17.8 17.7; 2 x 4096 x 640 14.6 13.1
// 11.9; 4 x 1140 x 960 11.5 12.9 11.2; 2 x 1024 x 1280 9.6 10.7 10.1; 2 x 411 x 1280 8.7 10.4 8.9; 1 x 337 x 320 7.5 8.2 7.6.
// Channels whose count is not a multiple of 8 take VEC = 2 (groups hold an even number of channels).
// ---------------------------------------------------------------------------------------
constexpr int GN_ITERS = 6;          // slabs of a workgroup that are in flight together
constexpr int GN_THREADS = 512, GN_MAX_THREADS = 1024;   // of a workgroup in both passes; the larger where one row needs it
constexpr int GN_TARGET_WGS = 256;   // partial-sum workgroups of a launch, one per CU, ...
constexpr int GN_MAX_PCHUNKS = 128;  // ... of a sample at most this many, ...
constexpr int GN_PSLABS = 4;         // ... and fewer rather than with fewer slabs
constexpr int GN_APPLY_WGS = 170;    // apply workgroups take more than one slab while this many are left (256: up to 8 % slower at 1 to 6 M elements)
constexpr int GN_EARLY_WGS = 600;    // second pass without SiLU: statistics requested ahead of the rows up to so many workgroups (groupnorm_apply_kernel)
constexpr int GN_RUN = 8;            // partials that a thread fetches together

template <int VEC>
struct GnVec;
template <>
struct GnVec<8> { typedef u32x4 type; };
template <>
struct GnVec<2> { typedef uint32_t type; };
template <int VEC>
__device__ __forceinline__ uint32_t gn_word(const typename GnVec<VEC>::type& v, int i) {
    if constexpr (VEC == 2) return v;
    else return v[i];
}

template <int VEC>
__global__ __launch_bounds__(GN_MAX_THREADS) void groupnorm_partial_kernel(const uint16_t* __restrict__ x, float* __restrict__ partials,
                                                                               int T, int C, int groups, int nchunks, int pchunk, int rows) {
    typedef typename GnVec<VEC>::type vec;
    constexpr int NP = VEC / 2;     // channel pairs of a thread
    extern __shared__ float sh[];   // [rows][C / 2] pair sums, two floats each
    const int b = blockIdx.y, chunk = blockIdx.x, tid = threadIdx.x;
    const int cpg = C / groups, nv = C / VEC, npairs = C >> 1;
    const int row = tid / nv, cv = tid - row * nv;
    const uint16_t* xb = x + (size_t)b * T * C;
    const int t1 = min(T, (chunk + 1) * pchunk);
    if (row < rows) {
        float s1[NP], s2[NP], shift[NP];
        int g0 = cv * VEC / cpg * cpg;       // first channel of the pair's group
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            s1[i] = s2[i] = 0.f;
            while (cv * VEC + 2 * i >= g0 + cpg) g0 += cpg;
            shift[i] = bf16_to_f32(xb[g0]);
        }
        for (int t = chunk * pchunk + row; t < t1; t += rows * GN_ITERS) {
            vec v[GN_ITERS];
#pragma unroll
            for (int k = 0; k < GN_ITERS; ++k)
                if (t + k * rows < t1) v[k] = reinterpret_cast<const vec*>(xb + (size_t)(t + k * rows) * C)[cv];
#pragma unroll
            for (int k = 0; k < GN_ITERS; ++k) {
                if (t + k * rows >= t1) break;
#pragma unroll
                for (int i = 0; i < NP; ++i) {
                    const uint32_t w = gn_word<VEC>(v[k], i);
                    const float a = bf16lo_to_f32(w) - shift[i], c = bf16hi_to_f32(w) - shift[i];
                    s1[i] += a + c;
                    s2[i] += a * a + c * c;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) *reinterpret_cast<float2*>(sh + 2 * ((size_t)row * npairs + cv * NP + i)) = make_float2(s1[i], s2[i]);
    }
    __syncthreads();
    for (int p = tid; p < npairs; p += blockDim.x) {   // tokens of a pair, in row order, into row 0
        float a1 = 0.f, a2 = 0.f;
#pragma unroll 4
        for (int r = 0; r < rows; ++r) {
            const float2 q = *reinterpret_cast<const float2*>(sh + 2 * ((size_t)r * npairs + p));
            a1 += q.x;
            a2 += q.y;
        }
        *reinterpret_cast<float2*>(sh + 2 * p) = make_float2(a1, a2);
    }
    __syncthreads();
    const int ppg = cpg >> 1;
    for (int g = tid; g < groups; g += blockDim.x) {
        float a1 = 0.f, a2 = 0.f;
#pragma unroll 4
        for (int i = 0; i < ppg; ++i) {
            const float2 q = *reinterpret_cast<const float2*>(sh + 2 * (g * ppg + i));
            a1 += q.x;
            a2 += q.y;
        }
        *reinterpret_cast<float2*>(partials + (((size_t)b * nchunks + chunk) * groups + g) * 2) = make_float2(a1, a2);
    }
}

// SILU: y = n * sigmoid(n) on the normalised value, the GroupNorm + SiLU pair of the base model's
// ResNet blocks as one operator (Section 4.3, "Kernel-level optimizations")
// EARLY: what the statistics and the affine need is requested ahead of the rows.  Loads come back in the order they are issued in: behind the rows of
// large inputs they take as long as those do (us with SiLU, inputs in turn from HBM, behind / ahead: 4 x 16384 x 320 30.9 / 28.7, 1 x 16384 x 1280 33.8 /
// 31.9, 2 x 16384 x 320 19.3 / 18.8, 4 x 1200 x 960 12.2 / 11.9; where a workgroup has few slabs the rows want to be first: 2 x 4096 x 320 10.2 / 10.4).
// Not without SiLU's arithmetic between loads and stores where workgroups follow each other on a CU (2 x 16384 x 320, 456 of them, 16.0 / 15.5; 1 x 43000 x 320,
// 598, 20.9 / 19.5; 9 x 1200 x 1280, 603, 19.7 / 19.8; 4 x 6200 x 640, 692, 20.3 / 20.8; 4 x 16384 x 320, 911, 24.3 / 25.3; 16 x 1024 x 1280, 912, 25.0 / 26.5),
// nor where a thread has 4 bytes of a row, six requests for eight or more ahead of them (1 x 12000 x 100 8.1 / 8.3, 8 x 3000 x 1220 45.2 / 48.0, with SiLU 8.5 / 8.6, 50.6 / 53.3).
// Batches of five samples and more have fewer partials to wait for, and a CU's first workgroup then waits longer for its rows than it did for those (20 x 900 x 320, 13
// partials, 260 workgroups, 12.1 / 12.8, with SiLU 14.6 / 14.9; 40 x 500 x 320 12.7 / 13.4, 15.0 / 15.4; 16 x 1600 x 320, 368, 13.9 / 14.1, 16.3 / 16.0; 90 x 300 x 320,
// 450, 14.9 / 14.7, 17.3 / 16.7; up to four samples all of 250 to 360 gain, 4 x 4610 x 320 13.1 / 12.7, 15.2 / 14.6).
template <int VEC, bool SILU, bool EARLY>
__global__ __launch_bounds__(GN_MAX_THREADS) void groupnorm_apply_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ y,
                                                                           const uint16_t* __restrict__ gamma, const uint16_t* __restrict__ beta,
                                                                           const float* __restrict__ partials, int T, int C, int groups, int nchunks,
                                                                           int parts, int rows, int iters, float eps) {
    typedef typename GnVec<VEC>::type vec;
    constexpr int NP = VEC / 2;
    extern __shared__ float sh[];   // [parts][groups] run sums, two floats each; then [groups] (mean, rstd)
    const int b = blockIdx.y, tid = threadIdx.x;
    const int cpg = C / groups, nv = C / VEC;
    const int row = tid / nv, cv = tid - row * nv;
    const uint16_t* xb = x + (size_t)b * T * C;
    uint16_t* yb = y + (size_t)b * T * C;
    const int t0 = blockIdx.x * rows * iters + row;
    const int t1 = min(T, (blockIdx.x + 1) * rows * iters);
    const bool mine = row < rows;
    // ---- statistics of the sample's groups.  A group's chunks are summed in `parts` contiguous runs
    // by as many threads, and the runs then in run order: a fixed order for a given shape
    const float2* src = reinterpret_cast<const float2*>(partials) + (size_t)b * nchunks * groups;
    float2* sub = reinterpret_cast<float2*>(sh);
    const int run = (nchunks + parts - 1) / parts, sums = parts * groups;
    float2 q[GN_RUN];
    auto fetch = [&](int i, int c) {      // run i's partials from its c-th on, all in flight together
        const int part = i / groups, last = min(nchunks, (part + 1) * run) - 1;
#pragma unroll
        for (int k = 0; k < GN_RUN; ++k) q[k] = src[(size_t)max(min(part * run + c + k, last), 0) * groups + (i - part * groups)];
    };
    float shift = 0.f;
    vec gv, bv;
    if (EARLY) {
        fetch(min(tid, sums - 1), 0);
        shift = bf16_to_f32(xb[min(tid, groups - 1) * cpg]);
        gv = reinterpret_cast<const vec*>(gamma)[mine ? cv : 0];
        bv = reinterpret_cast<const vec*>(beta)[mine ? cv : 0];
    }
    // this thread's inputs: they are in flight while the statistics are put together
    vec v[GN_ITERS];
#pragma unroll
    for (int k = 0; k < GN_ITERS; ++k)
        if (mine && t0 + k * rows < t1) v[k] = reinterpret_cast<const vec*>(xb + (size_t)(t0 + k * rows) * C)[cv];
    for (int i = tid; i < sums; i += blockDim.x) {
        float a1 = 0.f, a2 = 0.f;
        const int n = min(nchunks, (i / groups + 1) * run) - i / groups * run;
        for (int c = 0; c < n; c += GN_RUN) {
            if (!EARLY || i != tid || c) fetch(i, c);
#pragma unroll
            for (int k = 0; k < GN_RUN; ++k)
                if (c + k < n) { a1 += q[k].x; a2 += q[k].y; }
        }
        sub[i] = make_float2(a1, a2);
    }
    __syncthreads();
    float2* stat = sub + sums;
    for (int g = tid; g < groups; g += blockDim.x) {
        float a1 = 0.f, a2 = 0.f;
#pragma unroll 4
        for (int p = 0; p < parts; ++p) {
            a1 += sub[p * groups + g].x;
            a2 += sub[p * groups + g].y;
        }
        const float n = (float)T * (float)cpg;
        const float m1 = a1 / n;
        const float var = fmaxf(a2 / n - m1 * m1, 0.f);
        stat[g] = make_float2((EARLY && g == tid ? shift : bf16_to_f32(xb[g * cpg])) + m1, rsqrtf(var + eps));
    }
    __syncthreads();
    if (!mine) return;
    float mean[NP], g0[NP], g1[NP], b0[NP], b1[NP];
    if (!EARLY) {
        gv = reinterpret_cast<const vec*>(gamma)[cv];
        bv = reinterpret_cast<const vec*>(beta)[cv];
    }
    int g = cv * VEC / cpg;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        while (cv * VEC + 2 * i >= (g + 1) * cpg) ++g;
        const float2 q = stat[g];
        const uint32_t gw = gn_word<VEC>(gv, i), bw = gn_word<VEC>(bv, i);
        mean[i] = q.x;
        g0[i] = bf16lo_to_f32(gw) * q.y;
        g1[i] = bf16hi_to_f32(gw) * q.y;
        b0[i] = bf16lo_to_f32(bw);
        b1[i] = bf16hi_to_f32(bw);
    }
#pragma unroll
    for (int k = 0; k < GN_ITERS; ++k) {
        if (t0 + k * rows >= t1) break;
        vec o;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const uint32_t w = gn_word<VEC>(v[k], i);
            float o0 = (bf16lo_to_f32(w) - mean[i]) * g0[i] + b0[i];
            float o1 = (bf16hi_to_f32(w) - mean[i]) * g1[i] + b1[i];
            if (SILU) {
                o0 = o0 * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * o0));
                o1 = o1 * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * o1));
            }
            const bf16x2 pk = {(__bf16)o0, (__bf16)o1};
            if constexpr (VEC == 2) o = __builtin_bit_cast(uint32_t, pk);
            else o[i] = __builtin_bit_cast(uint32_t, pk);
        }
        reinterpret_cast<vec*>(yb + (size_t)(t0 + k * rows) * C)[cv] = o;
    }
}

// ---- one launch for samples that fit: a workgroup holds all tokens of a few groups (as many as fill whole 16-byte pieces of a
// row) in registers, so nothing has to be waited for across workgroups and x is read once.
//
// What bounds it: latency (launch, one round of loads, three barriers of the reduction) for short samples, and what one CU takes
// in and gives out for long ones, because there are only groups / unit workgroups to a sample and their pieces of a row are short.
// us with SiLU, two launches / this, by the rows that a thread holds: two 2 x 256 x 320 6.9 / 5.2, 1 x 337 x 320 6.9 / 5.3, one
// 2 x 64 x 1280 7.3 / 4.8, three 2 x 411 x 1280 9.1 / 7.1, five 4 x 300 x 960 8.9 / 8.5; six 2 x 1024 x 640 8.7 / 10.4,
// 2 x 1024 x 1280 10.4 / 10.7; eleven 2 x 2048 x 320 8.7 / 16.2.
constexpr int GN1_THREADS = 1024;
constexpr int GN1_MAX_ITERS = 4;
template <int ITERS, bool SILU>
__global__ __launch_bounds__(GN1_THREADS) void groupnorm_unit_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ y,
                                                                     const uint16_t* __restrict__ gamma, const uint16_t* __restrict__ beta,
                                                                     int T, int C, int cpg, int unit_groups, int units, float eps) {
    __shared__ float2 sh[GN1_THREADS * 4];      // [rows][pairs] sums of a thread's channel pairs
    __shared__ float2 part[GN1_THREADS];        // [pairs][parts] runs of rows
    __shared__ float2 stat[4];                  // (mean, rstd) of the unit's groups
    const int total = (int)gridDim.x;
    int wg = blockIdx.x;
    if ((total & 7) == 0) wg = (wg & 7) * (total >> 3) + (wg >> 3);     // neighbouring pieces of a row on one XCD
    const int b = wg / units, unit = wg - b * units, tid = threadIdx.x;
    const int nv = cpg * unit_groups >> 3, npairs = nv * 4, rows = GN1_THREADS / nv;
    const int row = tid / nv, cv = tid - row * nv;
    const bool mine = row < rows;
    const size_t at = (size_t)b * T * C + (size_t)unit * unit_groups * cpg;
    const uint16_t* const xb = x + at;
    u32x4 v[ITERS];
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
        v[k] = u32x4{0u, 0u, 0u, 0u};
        if (mine && row + k * rows < T) v[k] = reinterpret_cast<const u32x4*>(xb + (size_t)(row + k * rows) * C)[cv];
    }
    const int cg = unit * unit_groups * cpg / 8 + (mine ? cv : 0);
    const u32x4 gv = reinterpret_cast<const u32x4*>(gamma)[cg], bv = reinterpret_cast<const u32x4*>(beta)[cg];
    int grp[4];
    float shift[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        grp[i] = (cv * 8 + 2 * i) / cpg;
        shift[i] = bf16_to_f32(xb[grp[i] * cpg]);
    }
    if (mine) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int k = 0; k < ITERS; ++k)
                if (row + k * rows < T) {
                    const float a = bf16lo_to_f32(v[k][i]) - shift[i], c = bf16hi_to_f32(v[k][i]) - shift[i];
                    s1 += a + c;
                    s2 += a * a + c * c;
                }
            sh[row * npairs + cv * 4 + i] = make_float2(s1, s2);
        }
    }
    __syncthreads();
    const int used = min(rows, T), parts = GN1_THREADS / npairs;
    {
        const int p = tid % npairs, j = tid / npairs;
        if (j < parts) {
            float2 a = make_float2(0.f, 0.f);
            for (int r = j; r < used; r += parts) {
                const float2 q = sh[r * npairs + p];
                a.x += q.x;
                a.y += q.y;
            }
            part[p * parts + j] = a;
        }
    }
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63;
    if (wave < unit_groups) {
        const int ppg = cpg >> 1, n = ppg * parts;
        float2 a = make_float2(0.f, 0.f);
        for (int i = lane; i < n; i += 64) {
            const float2 q = part[wave * n + i];
            a.x += q.x;
            a.y += q.y;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            a.x += __shfl_xor(a.x, o);
            a.y += __shfl_xor(a.y, o);
        }
        if (lane == 0) {
            const float m = (float)T * (float)cpg;
            const float m1 = a.x / m;
            stat[wave] = make_float2(bf16_to_f32(xb[wave * cpg]) + m1, rsqrtf(fmaxf(a.y / m - m1 * m1, 0.f) + eps));
        }
    }
    __syncthreads();
    if (!mine) return;
    uint16_t* const yb = y + at;
    float mean[4], g0[4], g1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float2 q = stat[grp[i]];
        mean[i] = q.x;
        g0[i] = bf16lo_to_f32(gv[i]) * q.y;
        g1[i] = bf16hi_to_f32(gv[i]) * q.y;
    }
#pragma unroll
    for (int k = 0; k < ITERS; ++k) {
        if (row + k * rows >= T) break;
        u32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float o0 = (bf16lo_to_f32(v[k][i]) - mean[i]) * g0[i] + bf16lo_to_f32(bv[i]);
            float o1 = (bf16hi_to_f32(v[k][i]) - mean[i]) * g1[i] + bf16hi_to_f32(bv[i]);
            if (SILU) {
                o0 = o0 * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * o0));
                o1 = o1 * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896340736f * o1));
            }
            const bf16x2 pk = {(__bf16)o0, (__bf16)o1};
            o[i] = __builtin_bit_cast(uint32_t, pk);
        }
        reinterpret_cast<u32x4*>(yb + (size_t)(row + k * rows) * C)[cv] = o;
    }
}

// groups of a unit (0: two launches instead) and the rows that a thread of it holds.  Not where a unit's piece of a row is much
// less than a cache line, which every unit would fetch again, nor for batches that no longer fit the caches of the CUs at work.
static int gn_unit(int Bn, int T, int C, int groups, int* iters) {
    const int cpg = C / groups, unit = cpg % 8 == 0 ? 1 : cpg % 4 == 0 ? 2 : 4;
    const int nv = cpg * unit / 8;
    if (C % 8 || groups % unit || nv < 4 || nv * 4 > GN1_THREADS || (int64_t)Bn * T * C > (1 << 22)) return 0;
    const int rows = GN1_THREADS / nv;
    *iters = (T + rows - 1) / rows;
    return *iters <= GN1_MAX_ITERS ? unit : 0;
}
template <int ITERS>
static int launch_gn_unit(const uint16_t* x, uint16_t* y, const uint16_t* gamma, const uint16_t* beta, int Bn, int T, int C, int groups, int unit,
                          float eps, hipStream_t stream, bool silu) {
    const int units = groups / unit;
    if (silu) hipLaunchKernelGGL((groupnorm_unit_kernel<ITERS, true>), dim3(Bn * units), dim3(GN1_THREADS), 0, stream, x, y, gamma, beta, T, C, C / groups, unit, units, eps);
    else hipLaunchKernelGGL((groupnorm_unit_kernel<ITERS, false>), dim3(Bn * units), dim3(GN1_THREADS), 0, stream, x, y, gamma, beta, T, C, C / groups, unit, units, eps);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

size_t groupnorm_partials_bytes(int Bn, int T, int groups) {
    (void)T;
    return round_up((size_t)Bn * GN_MAX_PCHUNKS * groups * 2 * sizeof(float), 256);
}

template <int VEC>
static int launch_gn(const uint16_t* x, uint16_t* y, const uint16_t* gamma, const uint16_t* beta, int Bn, int T, int C, int groups, float eps,
                     float* partials, hipStream_t stream, bool silu) {
    const int nv = C / VEC;
    auto shape = [&](int most, int tokens, int* rows) {   // whole rows that fit `most` threads, no more than there are tokens
        *rows = most / nv;
        if (*rows > tokens) *rows = tokens;
        if (*rows < 1) *rows = 1;
        return (nv * *rows + 63) / 64 * 64;
    };
    // partial sums
    int want = (GN_TARGET_WGS + Bn - 1) / Bn;
    if (want > GN_MAX_PCHUNKS) want = GN_MAX_PCHUNKS;
    int prows, rows;
    const int most = nv > GN_THREADS ? GN_MAX_THREADS : GN_THREADS;
    const int pchunk = std::max((T + want - 1) / want, GN_PSLABS * (most / nv));   // short samples: a few slabs rather than more partials
    const int pthreads = shape(most, pchunk, &prows);
    const int nchunks = (T + pchunk - 1) / pchunk;
    const int athreads = shape(most, T, &rows);
    int parts = athreads / groups;
    if (parts > (nchunks + GN_RUN - 1) / GN_RUN) parts = (nchunks + GN_RUN - 1) / GN_RUN;
    if (parts < 1) parts = 1;
    const size_t lds = (size_t)(parts + 1) * groups * 2 * sizeof(float);
    // slabs per workgroup: all of them in flight for large inputs, fewer where that would leave CUs without a workgroup
    const int64_t slabs = (int64_t)Bn * ((T + rows - 1) / rows);
    const int iters = (int)std::min<int64_t>(GN_ITERS, std::max<int64_t>(1, slabs / GN_APPLY_WGS));
    const dim3 grid((T + rows * iters - 1) / (rows * iters), Bn);
    const int64_t wgs = (int64_t)grid.x * Bn;
    const bool early = VEC == 8 && iters == GN_ITERS && (silu || wgs <= GN_EARLY_WGS) && (nchunks >= 60 || wgs > (silu ? 300 : 400));
    if (SD_DRY_RUN("groupnorm%s; ", dry_detail(early ? ", statistics first" : ""))) return SD_OK;
    SD_REQUIRE(pthreads <= GN_MAX_THREADS, SD_EUNSUPPORTED, "groupnorm: C=%d", C);
    hipLaunchKernelGGL((groupnorm_partial_kernel<VEC>), dim3(nchunks, Bn), dim3(pthreads), (size_t)prows * C * sizeof(float), stream, x, partials, T, C,
                       groups, nchunks, pchunk, prows);
    SD_HIP_CHECK(hipGetLastError());
    auto apply = [&](auto with_silu, auto early) {
        hipLaunchKernelGGL((groupnorm_apply_kernel<VEC, decltype(with_silu)::value, decltype(early)::value>), grid, dim3(athreads), lds, stream, x, y, gamma, beta, partials, T, C, groups,
                           nchunks, parts, rows, iters, eps);
    };
    constexpr std::bool_constant<VEC == 8> ahead;
    if (silu && early) apply(std::true_type(), ahead);
    else if (silu) apply(std::true_type(), std::false_type());
    else if (early) apply(std::false_type(), ahead);
    else apply(std::false_type(), std::false_type());
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

int launch_groupnorm(const uint16_t* x, uint16_t* y, const uint16_t* gamma, const uint16_t* beta,
                     int Bn, int T, int C, int groups, float eps, float* partials, hipStream_t stream, bool silu) {
    SD_REQUIRE(groups > 0 && C % groups == 0 && (C / groups) % 2 == 0, SD_EUNSUPPORTED,
               "groupnorm: C=%d groups=%d (need an even number of channels per group)", C, groups);
    SD_REQUIRE(C <= 2048, SD_EUNSUPPORTED, "groupnorm: C=%d > 2048", C);
    if (Bn <= 0 || T <= 0) return SD_OK;
    int iters = 0;
    const int unit = gn_unit(Bn, T, C, groups, &iters);
    if (unit && SD_DRY_RUN("groupnorm unit; ")) return SD_OK;
    if (unit && iters <= 2) return launch_gn_unit<2>(x, y, gamma, beta, Bn, T, C, groups, unit, eps, stream, silu);
    if (unit) return launch_gn_unit<GN1_MAX_ITERS>(x, y, gamma, beta, Bn, T, C, groups, unit, eps, stream, silu);
    return C % 8 == 0 ? launch_gn<8>(x, y, gamma, beta, Bn, T, C, groups, eps, partials, stream, silu)
                      : launch_gn<2>(x, y, gamma, beta, Bn, T, C, groups, eps, partials, stream, silu);
}

}  // namespace sd
