// Flash-style attention for gfx950, head dim 64, no mask: softmax(q k^T / 8) v per
// (sample, head) without ever writing the scores (the transformer block's self-attention
// over the latent tokens and cross-attention to the text tokens).
//
// The kernel works on the TRANSPOSED score tile S^T = K Q^T: with the 16x16x32 bf16 MFMA
// the accumulator of lane l then holds one query (column l % 16) and four of the block's keys
// (rows), so the softmax row maximum is an in-register reduction plus exchanges between the four
// quads of 16 lanes, the running rescale factor is a per-lane
// scalar, and the exponentials of two key blocks, packed to bf16, are already laid out as the B operand of
// the second MFMA, O^T += V^T P^T.  V is consumed transposed ([C, keys]), which is how the
// v-projection GEMM writes it, so both K and V^T tiles are staged with 16-byte rows.
//
// What limits it: vector-ALU issue, at a clock that the chip lowers under load (1.8 to 1.95 GHz of 2.4).  Per 32 queries x 64 keys a SIMD
// issues 32 exponentials (8 clocks each, measured alone), 16 packings (4.5), 36 MFMAs (8.5), 16 LDS reads and four others (4), with plain keys 32 FMAs (4): 714
// and 842 clocks if none of it overlapped.  816 were measured with three wavefronts to a SIMD and plain keys, so little does, and the sum is no
// lower bound; that is the matrix core's 576.  LDS gives 256 bytes a clock and is asked for a sixth of it.  16x16x32 MFMAs, although two issues for one, because the 32x32x16 ones cost more energy and
// leave the row sums to instructions that do not run beside MFMAs: 12 x 4096 x 8 heads 426 -> 386 us, in a block of
// 2 x 4096 tokens of 640 channels 94 -> 86, 8 x 988 x 20 heads 58.6 -> 53.1.
//
// Workgroup: one group of 4 wavefronts, each owning 32 (or 64) queries, or two groups that share the key range; K / V^T tiles of 64 keys go from
// global memory straight into LDS rings (wave-wide 1 KB loads of XOR-swizzled 16-byte
// chunks), one tile ahead of the one being used.  K rows are placed in LDS with the keys
// of every 32-key group in the order [0-3, 8-11, 16-19, 24-27, 4-7, 12-15, 20-23, 28-31]: a lane's scores of two
// key blocks are then 8 consecutive keys, and the matching V^T operand is a
// single 16-byte LDS read of the plain [C, keys] layout.
//
// Work split.  A (sample, head, 128-query or 256-query tile) is a tile; a workgroup normally takes one (attention_plan).
// When the tile count lies between two and three per CU (640 tiles on 256 CUs leaves half
// the CUs with three tiles and half with two), the launch is padded to exactly three
// workgroups per CU by cutting the key range of the surplus tiles in half: every CU then
// holds two whole tiles and one half.  Where there are at most two tiles per CU and many keys,
// all tiles are cut (attention_nsplit).  The two halves of a cut tile leave their unnormalised
// accumulator, reference maximum and row sum in a scratch buffer and count themselves in on a
// per-tile counter; the half that arrives second merges the two inside the launch (without
// counters, a second, small kernel merges them).
#include "common.hpp"
#include "read_ahead.hpp"

namespace sd {

__device__ __forceinline__ int aswz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }
// which of a tile's 64 keys K row r of LDS holds: bits 4, 3, 2 of the key are bits 3, 2, 4 of the row
__device__ __forceinline__ int key_of_row(int r) { return (r & 35) | ((r & 12) << 1) | ((r & 16) >> 2); }

constexpr float RESCALE_LOG2 = 8.0f;

// where lanes of a direct-to-LDS load point when their V^T chunk lies past the padded keys
__device__ __attribute__((aligned(256))) uint32_t g_attn_zeros[64];

// one direct global -> LDS load: each lane fetches 16 bytes from its own address, the 64
// pieces land contiguously at LDS byte address `lds_base` (wave-uniform).  Completion is
// tracked by hand with vmcnt and a workgroup barrier.
__device__ __forceinline__ void attn_dma16(const void* gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(gptr) : "memory", "m0");
}
// same with a wave-uniform 64-bit base and a 32-bit unsigned byte offset per lane: the
// per-tile address arithmetic stays on the scalar unit
__device__ __forceinline__ void attn_dma16_so(const void* sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(voff), "s"(uniform_ptr(sbase)) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void attn_wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// One half of a cut tile: 32 accumulator values a thread, then its queries' reference maxima and row sums.  Cut tiles have 128 queries.
constexpr int PART_FLOATS = 34 * 256;

// Largest of what the four quads of a wavefront (16 lanes each) hold for the same query, in every lane: exchanges of rows
// of 16 lanes and of half-wavefronts
__device__ __forceinline__ float quads_max(float x) {
    float a = x, b = x, lo, hi;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    both_halves(fmaxf(a, b), lo, hi);
    return fmaxf(lo, hi);
}

// normalise and store: lane holds queries row + qb*16, d = (d0 + db)*16 + 4*quad + v; l: row sums, whole
template <int QB, int KD>
__device__ __forceinline__ void store_queries(const f32x4 (&o)[KD][QB], const float (&l)[QB], uint16_t* __restrict__ out, int64_t ldo,
                                              int b, int Tq, int row, int head, int d0, int quad) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float inv = 1.0f / l[qb];
        if (row + qb * 16 < Tq) {
            uint16_t* op = out + ((int64_t)b * Tq + row + qb * 16) * ldo + head * 64 + d0 * 16 + 4 * quad;
#pragma unroll
            for (int db = 0; db < KD; ++db) {
                bf16x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = (__bf16)(o[db][qb][e] * inv);
                *reinterpret_cast<bf16x4*>(op + db * 16) = w;
            }
        }
    }
}

// PRE: the keys arrive multiplied by 1/8 * log2(e) (the K projection's epilogue does it before
// rounding to bf16), so a score is already the exponent of 2, and the running reference maximum
// is subtracted by the matrix core: all rows of a lane's accumulator belong to its query, so they start at
// -m (one register, four times over) instead of 0, the accumulator holds
// s - m and the vector ALU only exponentiates.  Without PRE one FMA per score does both.
// The maximum of every half tile is measured and the
// reference moves whenever it is exceeded by 2^8.  With TRY (prescaled keys, and long
// ranges of plain ones) the kernel tries without first.  What
// the reference maximum is for is range, not accuracy: p = 2^(s - m) is formed, rounded and
// accumulated in floating point, whose relative precision does not depend on magnitude, so any m
// gives the same result as long as nothing overflows and the row sum does not vanish.  The first
// attempt therefore measures only a segment's first tile (m becomes a score that occurs: the row
// sum is >= 1 from then on); after it the exponentials are
// formed against that fixed reference with no maximum pass at all.  At the end every lane looks at
// its row sum and accumulator: if anything is not finite or close to it, some score lay 2^100 or more
// above the first tile's; a workgroup in which any wavefront saw that returns true without storing
// anything, and its caller runs the segment again in the measured form.
// nsplit == 0: workgroup i takes tile i.  Otherwise the grid holds nfull whole tiles (a multiple of 8) and
// 2 * nsplit half tiles, rounded up to a multiple of 8, dealt so that each XCD, and in dispatch order
// each CU, first receives its share of whole tiles and then its share of halves.
__host__ __device__ __forceinline__ int attention_grid(int nfull, int nsplit) { return nsplit ? nfull + (nsplit + 3) / 4 * 8 : nfull; }
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) int32_t lds_i32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;

typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

// QB: 16-query blocks of a wavefront.  GR: groups of four wavefronts; each takes an equal share of the key range for all of the
// workgroup's 64 * QB queries, and their states meet in LDS at the end.
// lds, per group: K [2][64 keys (permuted within 32)][8 chunks of 8 d], then V [2][64 d][8 chunks of 8 keys];  ml: [GR][2][64 * QB]
constexpr int ATTN_GROUP_CH = 4 * 512;   // 16-byte chunks
template <int QB, int GR, bool PRE, bool TRY>
__device__ __forceinline__ bool attention_body(const uint16_t* __restrict__ q, int64_t ldq,
                                               const uint16_t* __restrict__ k, int64_t ldk,
                                               const uint16_t* __restrict__ vt, int64_t ldvt,
                                               uint16_t* __restrict__ out, int64_t ldo,
                                               int Tq, int Tk, int Tkp, int heads, int qtiles, float c,
                                               int nfull, int nsplit, int total, float* __restrict__ parts, int32_t* __restrict__ arrived,
                                               lds_u32x4* const lds, lds_f32* const ml, lds_i32* const wg_redo, const int tid, const int bid, const bool again) {
    static_assert(TRY || !PRE, "scores formed with -m are not moved once the half before them has been looked at");
    constexpr int BQ = 64 * QB, KD = 4 / GR;
    constexpr int THREADS = 256 * GR;
    constexpr int PART = KD * QB * 4 * THREADS + 2 * BQ;     // floats of a part
    constexpr bool CUT = QB == 2;
    static_assert(!CUT || PART <= PART_FLOATS, "a part fits its share of the scratch memory");

    // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of
    // (sample, head, query tile) so that one head's K and V stay in one XCD's L2.
    const int nt = (Tk + 63) >> 6;
    int tile, s0 = 0, s1 = nt, part = -1;   // steps [s0, s1) of the tile; part >= 0: a half tile
    if (!CUT || nsplit == 0) {
        tile = bid;
        if ((total & 7) == 0) tile = (tile & 7) * (total >> 3) + (tile >> 3);
    } else {
        const int xcd = bid & 7, j = bid >> 3;
        const int fpx = nfull >> 3, hpx = (nsplit + 3) >> 2;   // whole tiles / halves per XCD
        if (j < fpx) {
            tile = xcd * fpx + j;
        } else {
            const int h = xcd * hpx + (j - fpx);
            if (h >= 2 * nsplit) return false;
            tile = nfull + (h >> 1);
            part = h & 1;
            const int mid = (nt + 1) >> 1;
            s0 = part ? mid : 0;
            s1 = part ? nt : mid;
        }
    }
    const int qt = tile % qtiles;
    const int head = (tile / qtiles) % heads, b = tile / (qtiles * heads);
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3, grp = GR == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8);
    const int l16 = lane & 15, quad = lane >> 4;
    const int q0 = qt * BQ + wave * 16 * QB;
    // this group's tiles are [g0, g0 + n), its keys end at kend: of an odd number of tiles the one in the middle is masked for the
    // first group, which sits out where it is the only one
    const int n = (s1 - s0 + GR - 1) / GR, g0 = GR > 1 && grp ? s1 - n : s0;
    const int kend = GR > 1 && grp == 0 ? (s1 - n) * 64 : min(Tk, s1 * 64);
    const bool live = g0 * 64 < kend;

    // ---- Q fragments (B operand of S^T = K Q^T): lane holds q[row l16][d = kk*32 + quad*8 ..+8]
    bf16x8 qf[QB][2];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        int row = q0 + qb * 16 + l16;
        row = row < Tq ? row : Tq - 1;
        const uint16_t* qp = q + ((int64_t)b * Tq + row) * ldq + head * 64 + quad * 8;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) qf[qb][kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qp + kk * 32));
    }

    // ---- tile loaders.  A tile is 8 blocks of 1 KB (8 rows x 8 chunks); load j of wave w
    // fills block j*4 + w: lane l lands at chunk position l % 8 of row l / 8 and fetches the
    // logical chunk the XOR swizzle places there.  K row r holds key key_of_row(r); keys past Tk
    // re-read the last key (masked later), V^T chunks past the padded key count read zeros.
    lds_u32x4* const ring = lds + grp * ATTN_GROUP_CH;
    const uint32_t ring_base = (uint32_t)(uintptr_t)ring;
    const uint16_t* kbase = k + (int64_t)b * Tk * ldk + head * 64;
    // rows of the two loads of a lane are 32 apart: same swizzled chunk for both
    const int r0 = wave * 8 + (lane >> 3);
    const int kc8 = aswz(r0, lane & 7) * 8;
    const int kkey0 = key_of_row(r0);
    // full tiles: byte offset of this lane's first K row and first V^T row from the tile's base; the
    // second row of each lies 32 rows further, a wave-uniform distance that goes into the scalar base
    const uint32_t koff = (uint32_t)(((int64_t)kkey0 * ldk + kc8) * 2);
    const uint32_t voff = (uint32_t)(((int64_t)r0 * ldvt + kc8) * 2);
    const int64_t krow32 = 64 * ldk, vrow32 = 64 * ldvt;     // bytes
    const char* vbase = reinterpret_cast<const char*>(vt + (int64_t)(head * 64) * ldvt + (int64_t)b * Tkp);
    auto issue_kv = [&](int t, int slot) {
        const int key0 = t * 64;
        const uint32_t kdst = ring_base + (uint32_t)(slot * 8192 + wave * 1024);
        const uint32_t vdst = kdst + 16384;
        if (key0 + 64 > Tk) {
            // (the lane's row and chunk are derived afresh from a laundered lane index, so that
            // nothing of this rare path is kept in registers through the key loop)
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int rr = wave * 8 + (ln >> 3);
            const int cc8 = aswz(rr, ln & 7) * 8;
            const int kk0 = key_of_row(rr);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                int key = key0 + kk0 + j * 32;
                key = key < Tk ? key : Tk - 1;
                attn_dma16(kbase + (int64_t)key * ldk + cc8, kdst + j * 4096);
            }
            const bool inside = key0 + cc8 < Tkp;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const void* src = inside ? (const void*)(vbase + key0 * 2 + ((int64_t)(rr + j * 32) * ldvt + cc8) * 2) : (const void*)g_attn_zeros;
                attn_dma16(src, vdst + j * 4096);
            }
        } else {
            const char* kb = reinterpret_cast<const char*>(kbase) + (int64_t)key0 * ldk * 2;
            const char* vb = vbase + key0 * 2;
#pragma unroll
            for (int j = 0; j < 2; ++j) attn_dma16_so(kb + j * krow32, koff, kdst + j * 4096);
#pragma unroll
            for (int j = 0; j < 2; ++j) attn_dma16_so(vb + j * vrow32, voff, vdst + j * 4096);
        }
    };

    constexpr bool KEEP_M = PRE && QB == 2;      // -m ready as the start of the scores (registers)
    f32x4 o[4][QB], ls[QB], mneg[KEEP_M ? QB : 1];
    float m[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        if (KEEP_M) mneg[KEEP_M ? qb : 0] = f32x4{0.f, 0.f, 0.f, 0.f};
        m[qb] = PRE && live ? 0.f : -INFINITY;
        ls[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int db = 0; db < 4; ++db) o[db][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // A key tile is worked through in halves of 32 keys: scores of one half while the half before is exponentiated.
    // Rows that are 16 apart share the swizzle.
    const int lrow8 = l16 * 8, lsw = (l16 >> 1) & 7;
    // K fragments of half h: kf[kb][kk], key block kb, d = kk*32 ..
    auto load_kfrags = [&](int slot, int h, bf16x8 (&kf)[2][2]) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const lds_u32x4* lk = ring + slot * 512 + h * 256 + lrow8 + ((kk * 4 + quad) ^ lsw);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) kf[kb][kk] = __builtin_bit_cast(bf16x8, lk[kb * 128]);
        }
    };
    // With the K row order above, a lane's scores of a half are its keys quad*8 ..+8, the 16-byte chunk h*4 + quad of a V^T row
    auto load_vfrags = [&](int slot, int h, bf16x8 (&vf)[4]) {
        const lds_u32x4* lv = ring + 1024 + slot * 512 + lrow8 + ((h * 4 + quad) ^ lsw);
#pragma unroll
        for (int db = 0; db < 4; ++db) vf[db] = __builtin_bit_cast(bf16x8, lv[db * 128]);
    };
    // scores of a half; all of a lane's accumulator values belong to its query, so they can start at -m
    auto compute_s = [&](f32x4 (&s)[2][QB], bf16x8 (&kf)[2][2]) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const float x = PRE ? -m[qb] : 0.f;
                s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][0], qf[qb][0], KEEP_M ? mneg[KEEP_M ? qb : 0] : f32x4{x, x, x, x}, 0, 0, 0);
            }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][1], qf[qb][1], s[kb][qb], 0, 0, 0);
    };
    // a group's last tile: keys from kend on get a score of -inf, and their values (padding holds whatever the
    // caller's buffer held) become zeros, so that 0 * garbage stays 0
    auto mask_scores = [&](int t, int h, f32x4 (&s)[2][QB]) {
        const int left = kend - (t * 64 + h * 32 + quad * 8);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (kb * 4 + v >= left) {
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) s[kb][qb][v] = -INFINITY;
                }
    };
    auto mask_values = [&](int t, int h, bf16x8 (&vf)[4]) {
        const int left = kend - (t * 64 + h * 32 + quad * 8);
        u32x4 keep;
#pragma unroll
        for (int i = 0; i < 4; ++i) keep[i] = 2 * i + 1 < left ? 0xffffffffu : 2 * i < left ? 0xffffu : 0u;
#pragma unroll
        for (int db = 0; db < 4; ++db) vf[db] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, vf[db]) & keep);
    };
    // Running-maximum bookkeeping of a half: the reference maximum m only moves when a
    // score exceeds it by more than RESCALE_LOG2 in the exponent (p <= 2^RESCALE_LOG2
    // stays far inside fp32 / bf16 range), so the O and row sum rescale runs on the first tiles and
    // almost never afterwards.  This lane's queries are column l16 of each block, its keys are its registers; it looks at those alone
    // (`over`), and any lane over the limit has all quads look together.
    // PRE: the scores arrive already shifted by m, so their maximum is the excess over it.  The first tile always sets the reference (m starts at 0,
    // not at the scores' level).
    auto lane_max = [&](f32x4 (&s)[2][QB], int qb) {
        float mx = fmaxf(s[0][qb][0], s[1][qb][0]);
#pragma unroll
        for (int v = 1; v < 4; ++v) mx = fmaxf(fmaxf(mx, s[0][qb][v]), s[1][qb][v]);
        return mx;
    };
    auto over = [&](float mx, int qb) { return PRE ? mx > RESCALE_LOG2 : (mx - m[qb]) * c > RESCALE_LOG2; };
    auto move_max = [&](int qb, float lane_mx, f32x4 (&s)[2][QB], bool first) {
        // the other quads hold the other keys of this query: lane swaps (vector-ALU operations, no LDS round trip)
        const float mx = quads_max(lane_mx);
        // Nothing has been summed up when the reference is first set, so nothing is rescaled: for scores below -128 the factor would be
        // infinite, and infinity times the sums' zeros NaN.
        // A tile of nothing but -inf weighs nothing; its reference is one that any score exceeds.  (PRE: the scores start at -m, and a huge one would
        // swallow them.  So it is 0, and where everything behind that tile lies so far below that the row sum vanishes, the second attempt starts at -2^13, from
        // where fp32 still resolves 2^-10.  What lies 2^126 and more below that counts for nothing.)
        if (first) {
            m[qb] = PRE ? (mx == -INFINITY ? (again ? -8192.f : 0.f) : mx) : fmaxf(mx, -3.4028234663852886e38f);
            if (KEEP_M) mneg[KEEP_M ? qb : 0] = f32x4{-m[qb], -m[qb], -m[qb], -m[qb]};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                if (PRE) s[kb][qb] -= m[qb];
            return;
        }
        float alpha;
        if (PRE) {
            const float delta = mx > RESCALE_LOG2 ? mx : 0.f;
            alpha = __builtin_amdgcn_exp2f(-delta);
            m[qb] += delta;
            if (KEEP_M) mneg[KEEP_M ? qb : 0] = f32x4{-m[qb], -m[qb], -m[qb], -m[qb]};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) s[kb][qb] -= delta;
        } else {
            const float mnew = over(mx, qb) ? mx : m[qb];
            alpha = __builtin_amdgcn_exp2f((m[qb] - mnew) * c);
            m[qb] = mnew;
        }
        ls[qb] *= alpha;
#pragma unroll
        for (int db = 0; db < 4; ++db) o[db][qb] *= alpha;
    };
    // The second attempt looks before it forms the probabilities.
    auto look_first = [&](f32x4 (&s)[2][QB]) {
        if (!TRY || !again) return;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float mx = lane_max(s, qb);
            if (__builtin_amdgcn_ballot_w64(over(mx, qb)) != 0ull) move_max(qb, mx, s, false);
        }
    };
    // p = exp2((s - m) * c) packed to bf16 in MFMA operand order
    auto exponentials = [&](f32x4 (&s)[2][QB], bf16x8 (&pf)[QB]) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float mc = m[qb] * c;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 4; ++v) pf[qb][kb * 4 + v] = (__bf16)__builtin_amdgcn_exp2f(PRE ? s[kb][qb][v] : s[kb][qb][v] * c - mc);
        }
    };
    // Kernels that measure every tile look afterwards, beside the exponentials, and form the probabilities once more where a
    // score lies too far above the reference: 8 x 988 x 20 heads 54.4 -> 53.6 us, 8 x 512 x 10 14.5 -> 14.0.
    auto look_after = [&](f32x4 (&s)[2][QB], bf16x8 (&pf)[QB]) {
        if (TRY) return;
        float mx[QB];
        bool need = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            mx[qb] = lane_max(s, qb);
            need = need || over(mx[qb], qb);
        }
        if (__builtin_amdgcn_ballot_w64(need) == 0ull) return;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) move_max(qb, mx[qb], s, false);
        exponentials(s, pf);
    };
    // O^T += V^T P^T.  The row sums are one more block of rows, of ones: the normaliser matches exactly what is multiplied,
    // every lane has its queries' whole sums, and the vector ALU does nothing for them.  (v_dot2c_f32_bf16, which adds up two
    // a lane, does not run beside MFMAs: 32 exponentials, 16 packings and 32 MFMAs take 593 clocks of a SIMD, 786 with 16 of those among them.)
    u32x4 ones_bits = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    asm volatile("" : "+v"(ones_bits));
    const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);
    auto accumulate_o = [&](bf16x8 (&vf)[4], bf16x8 (&pf)[QB]) {
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) o[db][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[db], pf[qb], o[db][qb], 0, 0, 0);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) ls[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[qb], ls[qb], 0, 0, 0);
    };

    // ---- prologue: the first two key tiles in flight, scores of the first tile
    if (live) {
        issue_kv(g0, 0);
        if (n > 1) {
            issue_kv(g0 + 1, 1);
            attn_wait_vmcnt<4>();
        } else {
            attn_wait_vmcnt<0>();
        }
    }
    __syncthreads();
    const int last = g0 + n - 1;
    const bool masked = last * 64 + 64 > kend;
    f32x4 sa[2][QB], sb[2][QB];
    bf16x8 kf[2][2], vf[4], pf[QB];
    if (live) {
        // The first tile sets the reference, its second half too (formed once more in its turn): a query's largest weight is then mostly
        // 1, which bf16 holds exactly.  Set by the first half alone, 2 x 4096 x 10 heads on 77 keys were 2.6 % further from float64.
        load_kfrags(0, 1, kf);
        compute_s(sb, kf);
        if (n == 1 && masked) mask_scores(last, 1, sb);
        float mx[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) mx[qb] = lane_max(sb, qb);
        load_kfrags(0, 0, kf);
        compute_s(sa, kf);
        if (n == 1 && masked) mask_scores(last, 0, sa);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) move_max(qb, fmaxf(mx[qb], lane_max(sa, qb)), sa, true);
    }

    // ---- main loop, software-pipelined: the score MFMAs of one half are independent of the exponentials of the half before
    // and sit in the same basic block, so the matrix pipe and the vector ALU overlap inside one wavefront.
    // At the edge between two tiles the last of the old one's operands are in registers: when this wavefront's loads of the new
    // one have landed, one barrier says that it is whole and the slot of the old one free, which takes the tile after next.
#pragma unroll 1
    for (int i = 0; i + 1 < n; ++i) {
        const int slot = i & 1;
        load_kfrags(slot, 1, kf);
        load_vfrags(slot, 0, vf);
        __builtin_amdgcn_sched_barrier(0);
        look_first(sa);
        compute_s(sb, kf);
        exponentials(sa, pf);
        look_after(sa, pf);
        accumulate_o(vf, pf);
        load_vfrags(slot, 1, vf);
        attn_wait_vmcnt<0>();
        __syncthreads();
        if (i + 2 < n) issue_kv(g0 + i + 2, slot);
        load_kfrags(slot ^ 1, 0, kf);
        __builtin_amdgcn_sched_barrier(0);
        look_first(sb);
        compute_s(sa, kf);
        exponentials(sb, pf);
        look_after(sb, pf);
        accumulate_o(vf, pf);
    }
    if (live) {
        const int slot = (n - 1) & 1;
        if (n > 1 && masked) mask_scores(last, 0, sa);
        load_kfrags(slot, 1, kf);
        load_vfrags(slot, 0, vf);
        look_first(sa);
        compute_s(sb, kf);
        if (masked) {
            mask_values(last, 0, vf);
            mask_scores(last, 1, sb);
        }
        exponentials(sa, pf);
        look_after(sa, pf);
        accumulate_o(vf, pf);
        look_first(sb);
        load_vfrags(slot, 1, vf);
        if (masked) mask_values(last, 1, vf);
        exponentials(sb, pf);
        look_after(sb, pf);
        accumulate_o(vf, pf);
    }

    if (TRY && !again) {
        // did the attempt stay in range?  (a row sum of +inf, or NaN anywhere, says no.)  The limit leaves room for
        // what the tail adds up: the sums of two groups of two halves of a cut tile must stay finite, and the
        // reciprocal of theirs a normal number.
        // Prescaled keys: a row sum below 1 says that the reference was not a score (a first tile of -inf).
        float mag = 0.f;
        bool low = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            mag += ls[qb][0];
            if (PRE && live) low = low || ls[qb][0] < 0x1p-60f;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int v = 0; v < 4; ++v) mag += fabsf(o[db][qb][v]);
        }
        const bool bad = __builtin_amdgcn_ballot_w64(low || !(mag <= 1.0e37f)) != 0ull;
        if (bad && lane == 0) *wg_redo = 1;
    }
    if ((TRY && !again) || GR > 1) __syncthreads();     // (which also ends every wavefront's reads of the tiles)
    if (TRY && !again && __builtin_expect(__builtin_amdgcn_readfirstlane(*wg_redo) != 0, 0)) return true;

    // the scores are in score units, or already in exponent units when the keys were prescaled
    const float cm = PRE ? 1.0f : c;
    float l[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        l[qb] = ls[qb][0];
        if (PRE) m[qb] = l[qb] == 0.f ? -INFINITY : m[qb];     // (no key of weight in this range: the reference was none)
    }
    // ---- the groups' states about their common maximum: each finishes KD of the four d blocks
    f32x4 fin[KD][QB];
    if constexpr (GR == 1) {
#pragma unroll
        for (int db = 0; db < KD; ++db)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) fin[db][qb] = o[db][qb];
    } else {
        lds_f32x4* const ex = reinterpret_cast<lds_f32x4*>(lds) + (tid & 255);
#pragma unroll
        for (int db = 0; db < KD; ++db)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                ex[grp * ATTN_GROUP_CH + (db * QB + qb) * 256] = grp ? o[db][qb] : o[KD + db][qb];
                fin[db][qb] = grp ? o[KD + db][qb] : o[db][qb];
            }
        lds_f32* const mq = ml + wave * 16 * QB + l16;
        if (quad == 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                mq[grp * 2 * BQ + qb * 16] = m[qb];
                mq[(grp * 2 + 1) * BQ + qb * 16] = l[qb];
            }
        }
        __syncthreads();
        const int og = grp ^ 1;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float mo = mq[og * 2 * BQ + qb * 16], lo = mq[(og * 2 + 1) * BQ + qb * 16];
            const float mm = fmaxf(m[qb], mo);
            const float fs = __builtin_amdgcn_exp2f((m[qb] - mm) * cm), fo = __builtin_amdgcn_exp2f((mo - mm) * cm);
            const float f0 = grp ? fo : fs, f1 = grp ? fs : fo;      // the first group's term, then the second's, in both
            l[qb] = (grp ? lo : l[qb]) * f0 + (grp ? l[qb] : lo) * f1;
            m[qb] = mm;
#pragma unroll
            for (int db = 0; db < KD; ++db) {
                const f32x4 ov = ex[og * ATTN_GROUP_CH + (db * QB + qb) * 256];
#pragma unroll
                for (int v = 0; v < 4; ++v) fin[db][qb][v] = (grp ? ov[v] : fin[db][qb][v]) * f0 + (grp ? fin[db][qb][v] : ov[v]) * f1;
            }
        }
    }

    // ---- a whole tile is normalised and stored; half of a cut tile leaves its state behind
    if (!CUT || part < 0) {
        store_queries(fin, l, out, ldo, b, Tq, q0 + l16, head, grp * KD, quad);
        return false;
    }
    float* const pp = parts + ((size_t)(tile - nfull) * 2 + part) * PART;
    float* const pm = pp + KD * QB * 4 * THREADS + wave * 16 * QB + l16;    // maxima, sums BQ further: one quad of the first group writes them
    if (!arrived) {
#pragma unroll
        for (int db = 0; db < KD; ++db)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int v = 0; v < 4; ++v) pp[((db * QB + qb) * 4 + v) * THREADS + tid] = fin[db][qb][v];
        if (grp == 0 && quad == 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) pm[qb * 16] = m[qb], pm[BQ + qb * 16] = l[qb];
        }
        return false;
    }
    // Merge inside the launch: both halves leave their state (device-scope stores: the other
    // half may run on another XCD), then count themselves in; the one that arrives second
    // reads the first one's state and finishes the tile.  Nobody waits.  The counter is
    // zero before the launch and the second arrival puts it back.
    const int cut = tile - nfull;
    auto put = [](float* p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto get = [](const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
#pragma unroll
    for (int db = 0; db < KD; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int v = 0; v < 4; ++v) put(pp + ((db * QB + qb) * 4 + v) * THREADS + tid, fin[db][qb][v]);
    if (grp == 0 && quad == 0) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) put(pm + qb * 16, m[qb]), put(pm + BQ + qb * 16, l[qb]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // a device-scope store counts until it is visible at that scope
    __syncthreads();                                    // ... for every wave of this half; LDS is free from here on
    lds_i32* const first = reinterpret_cast<lds_i32*>(lds);
    if (tid == 0) *first = __hip_atomic_fetch_add(arrived + cut, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*first == 1) {
        if (tid == 0) __hip_atomic_store(arrived + cut, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const ptrdiff_t other = (part ? -1 : 1) * (ptrdiff_t)PART;
        float f0[QB], f1[QB], lsum[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float mo = get(pm + other + qb * 16), lo = get(pm + other + BQ + qb * 16);
            const float mm = fmaxf(m[qb], mo);
            const float fs = __builtin_amdgcn_exp2f((m[qb] - mm) * cm), fo = __builtin_amdgcn_exp2f((mo - mm) * cm);
            // same expression, operand for operand, whichever half arrives second: first half's term, then second's
            f0[qb] = part == 0 ? fs : fo, f1[qb] = part == 0 ? fo : fs;
            lsum[qb] = (part == 0 ? l[qb] : lo) * f0[qb] + (part == 0 ? lo : l[qb]) * f1[qb];
        }
#pragma unroll
        for (int db = 0; db < KD; ++db)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float ov = get(pp + other + ((db * QB + qb) * 4 + v) * THREADS + tid);
                    const float a0 = part == 0 ? fin[db][qb][v] : ov, a1 = part == 0 ? ov : fin[db][qb][v];
                    fin[db][qb][v] = a0 * f0[qb] + a1 * f1[qb];
                }
        store_queries(fin, lsum, out, ldo, b, Tq, q0 + l16, head, grp * KD, quad);
    }
    return false;
}

template <int QB, int GR, bool PRE, bool TRY, bool AHEAD>
__global__ __launch_bounds__(256 * GR, GR == 1 && QB == 2 ? 3 : 2) void attention_kernel(const uint16_t* __restrict__ q, int64_t ldq,
                                                        const uint16_t* __restrict__ k, int64_t ldk,
                                                        const uint16_t* __restrict__ vt, int64_t ldvt,
                                                        uint16_t* __restrict__ out, int64_t ldo,
                                                        int Tq, int Tk, int Tkp, int heads, int qtiles, float c,
                                                        int nfull, int nsplit, float* __restrict__ parts, int32_t* __restrict__ arrived,
                                                        const std::conditional_t<AHEAD, ReadRanges, NoRanges> ra) {
    const int total = AHEAD ? attention_grid(nfull, nsplit) : (int)gridDim.x;
    if constexpr (AHEAD) {
        // (the arguments in one batch, not a second one behind the branch)
        asm volatile("" ::"s"(q), "s"(ldq), "s"(k), "s"(ldk), "s"(vt), "s"(ldvt), "s"(Tq), "s"(Tk), "s"(Tkp), "s"(heads), "s"(qtiles));
        if ((int)blockIdx.x >= total) {
            read_ahead<16>(ra, ((int)blockIdx.x - total) * GR + (int)(threadIdx.x >> 8), (int)threadIdx.x & 255);
            return;
        }
    }
    __shared__ u32x4 tiles[GR * ATTN_GROUP_CH];
    __shared__ float maxima[GR == 1 ? 1 : GR * 2 * 64 * QB];
    __shared__ int32_t wg_redo;         // some wavefront's unmeasured attempt overflowed
    lds_u32x4* const lk = (lds_u32x4*)tiles;
    lds_f32* const ml = (lds_f32*)maxima;
    lds_i32* const redo = (lds_i32*)&wg_redo;
    if (TRY && threadIdx.x == 0) *redo = 0;    // (ordered before its first use by the key loop's barriers)
    // (One body for both attempts: as two, the second one's values took registers from the first, 65 to 150 of them spilled.  The second trip's
    // indexes are opaque: what both trips form of them would be formed ahead of the loop and kept, 64 queries to a wavefront spilled 44 registers in one
    // group.  In two groups they spill nothing and are faster so: 1 x 4096 x 10 heads 67.6 us, 68.4 with opaque ones.)
    bool again = false;
    int tid = threadIdx.x, bid = blockIdx.x;
    while (attention_body<QB, GR, PRE, TRY>(q, ldq, k, ldk, vt, ldvt, out, ldo, Tq, Tk, Tkp, heads, qtiles, c, nfull, nsplit, total, parts, arrived, lk, ml, redo,
                                            tid, bid, again)) {
        again = true;
        if constexpr (QB == 2 || GR == 1) asm volatile("" : "+v"(tid), "+s"(bid));
    }
}

// One workgroup per cut tile: combine the two halves about their common maximum.  Threads as in the kernel that left them.
template <int QB, int GR>
__global__ __launch_bounds__(256 * GR) void attention_merge_kernel(const float* __restrict__ parts, uint16_t* __restrict__ out, int64_t ldo,
                                                              int Tq, int heads, int qtiles, int nfull, float c) {
    constexpr int BQ = 64 * QB, KD = 4 / GR, THREADS = 256 * GR, PART = KD * QB * 4 * THREADS + 2 * BQ;
    const int tile = nfull + blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = (tid >> 6) & 3, grp = tid >> 8;
    const int l16 = lane & 15, quad = lane >> 4;
    const float* pa = parts + ((size_t)blockIdx.x * 2) * PART;
    const float* pb = pa + PART;
    const int at = KD * QB * 4 * THREADS + wave * 16 * QB + l16;
    f32x4 o[KD][QB];
    float l[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float ma = pa[at + qb * 16], mb = pb[at + qb * 16];
        const float mm = fmaxf(ma, mb);
        const float fa = __builtin_amdgcn_exp2f((ma - mm) * c), fb = __builtin_amdgcn_exp2f((mb - mm) * c);
#pragma unroll
        for (int db = 0; db < KD; ++db)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = ((db * QB + qb) * 4 + v) * THREADS + tid;
                o[db][qb][v] = pa[i] * fa + pb[i] * fb;
            }
        l[qb] = pa[at + BQ + qb * 16] * fa + pb[at + BQ + qb * 16] * fb;
    }
    const int qt = tile % qtiles;
    const int head = (tile / qtiles) % heads, b = tile / (qtiles * heads);
    store_queries(o, l, out, ldo, b, Tq, qt * BQ + wave * 16 * QB + l16, head, grp * KD, quad);
}

// CUs of the current device (cached; the query allocates nothing)
static int device_cus() {
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cus[dev] = n;
    }
    return cus[dev];
}

// number of tiles to cut in half (0: one workgroup per tile)
// block: inside an attention block, where the halves are merged in the launch.  Up to two tiles per CU and from 24 key tiles on, all
// are cut there if the most loaded CU then has less to do, and from 48 on also one per CU.  (us, a whole self-attention block without adapters, whole tiles of
// whatever kernel attention_plan has for them / cut: 1 x 1500 x 640 channels 39.6 / 36.7, 1 x 2048 x 1280 83.2 / 77.7, 1 x 3952 x 640 102.9 / 89.9, 1 x 4096 x 640
// 102.1 / 88.8, 2 x 4096 x 320 102.1 / 87.0, 1 x 3000 x 320 46.8 / 39.5, 2 x 2048 x 640 73.6 / 67.7; with as much on a CU as before 1 x 1500 x 1280
// 59.7 / 62.9, 1 x 2048 x 640 43.9 / 46.1, 1 x 2500 x 640 51.6 / 54.5, 1 x 4096 x 960 132.6 / 132.6, 2 x 3000 x 320 56.7 / 59.3.
// One per CU: 1 x 3952 x 320 51.4 / 55.0, 1 x 4096 x 320 52.8 / 55.4, 1 x 3840 x 512 61.5 / 64.6.  That line was drawn when a whole tile had one
// group of wavefronts, 63.3 / 57.3 at 4096 x 320; with two it no longer pays.  At 16 key tiles, before there were two groups: 2 x 988 x 640 38.8 / 39.1,
// 1 x 1024 x 1280 44.0 / 45.6.)
static int attention_nsplit(int Bn, int Tq, int Tk, int heads, bool block) {
    const long tiles = (long)((Tq + 127) / 128) * heads * Bn;
    const int nt = (Tk + 63) / 64;
    const long cus = device_cus();
    if (block && nt >= 24 && tiles <= 2 * cus && ((nt >= 48 && tiles <= cus) || (2 * tiles + cus - 1) / cus < 2 * ((tiles + cus - 1) / cus))) return (int)tiles;
    if (nt < 8 || tiles <= 2 * cus || tiles >= 3 * cus) return 0;
    const long nsplit = 3 * cus - tiles, nfull = tiles - nsplit;
    if (nfull <= 0 || (nfull & 7) || (nsplit & 3)) return 0;
    return (int)nsplit;
}

size_t attention_scratch_bytes(int Bn, int Tq, int Tk, int heads, bool block) {
    if (Bn <= 0 || Tq <= 0 || Tk <= 0 || heads <= 0) return 0;
    return (size_t)attention_nsplit(Bn, Tq, Tk, heads, block) * 2 * PART_FLOATS * sizeof(float);
}

// Which kernel, and its tiles: whole ones, and ones whose key range is cut in half (nsplit of them; 128 queries each, as the scratch
// memory is laid out for).
//   Up to one tile of 128 queries per CU the workgroup's key range goes to two groups of wavefronts, from eight key tiles on (us,
// standalone, one group / two: 1 x 1024 x 20 heads 17.5 / 15.4, 1 x 4096 x 5 50.5 / 41.0, 1 x 512 x 5 10.2 / 9.6, 2 x 256 x 10 8.4 / 8.5); cut tiles
// too, where their halves are one per CU.  Each group takes half of the tiles, rounded up, so few and odd ones gain least: 2 x 10 heads, both with the
// attempt without maxima, 576 keys 10.1 / 10.9, 640 10.8 / 10.6, 704 11.5 / 11.9, 768 12.2 / 11.8, 832 13.3 / 13.7, 896 14.1 / 13.6.
//   Tiles of 256 queries, 64 to a wavefront, read K and V^T half as often, but few of them load the CUs unevenly, and two wavefronts
// to a SIMD is all that the registers hold.  With two groups of wavefronts where they are one round (128 / 256 queries: 1 x 4096 x 10 71.3 / 65.9,
// 2 x 2500 x 10 47.5 / 44.9, 2 x 1500 x 20 31.6 / 31.0, 2 x 1024 x 20 23.9 / 25.6), with one where rounds of them come out ahead (4 x 3000 x 10 105 / 98,
// 4 x 4096 x 20 331 / 311, 8 x 1500 x 20 106 / 102; 2 x 4096 x 20, three rounds for five of the small ones, 171 / 189).
struct AttnPlan { int qb, gr, qtiles, nfull; };
static AttnPlan attention_plan(int Bn, int Tq, int nt, int heads, int nsplit) {
    AttnPlan p;
    const long cus = device_cus(), tiles = (long)((Tq + 127) / 128) * heads * Bn, wide = (long)((Tq + 255) / 256) * heads * Bn;
    p.qb = 2;
    p.gr = (nsplit > 0 ? tiles <= cus / 2 : tiles <= cus && nt >= 8) ? 2 : 1;
    if (nsplit == 0 && tiles > cus && wide <= cus && nt >= 24) p.qb = 4, p.gr = 2;
    if (nsplit == 0 && wide > cus && nt >= 20 && (double)((wide + cus - 1) / cus) * 1.85 < (double)((tiles + cus - 1) / cus)) p.qb = 4;
    p.qtiles = (Tq + 64 * p.qb - 1) / (64 * p.qb);
    p.nfull = p.qtiles * heads * Bn - nsplit;
    return p;
}

int launch_attention(const uint16_t* q, int64_t ldq, const uint16_t* k, int64_t ldk,
                     const uint16_t* vt, int64_t ldvt, uint16_t* out, int64_t ldo,
                     int Bn, int Tq, int Tk, int Tkp, int heads, bool k_prescaled, void* scratch, size_t scratch_bytes, int* cut_tiles,
                     hipStream_t stream, int32_t* arrived, int arrived_n, ReadAhead* ahead) {
    SD_REQUIRE(q && k && vt && out, SD_EINVAL, "attention: null pointer");
    SD_REQUIRE(Tk >= 1 && Tkp >= Tk && Tkp % 8 == 0, SD_EINVAL, "attention: Tk=%d Tkp=%d", Tk, Tkp);
    SD_REQUIRE(ldq % 8 == 0 && ldk % 8 == 0 && ldvt % 8 == 0 && ldo % 4 == 0, SD_EINVAL, "attention: leading dimensions");
    SD_REQUIRE(ldk > 0 && ldvt > 0 && ldk < (1 << 23) && ldvt < (1 << 23), SD_EINVAL, "attention: leading dimensions out of range");
    *cut_tiles = 0;
    if (Bn <= 0 || Tq <= 0 || heads <= 0) return SD_OK;
    const float c = 0.125f * 1.44269504088896340736f;   // 1/sqrt(64) * log2(e)
    SD_REQUIRE((long)((Tq + 127) / 128) * heads * Bn < (1l << 30), SD_EINVAL, "attention: problem too large");
    int nsplit = attention_nsplit(Bn, Tq, Tk, heads, k_prescaled);
    const size_t need = (size_t)nsplit * 2 * PART_FLOATS * sizeof(float);
    if (nsplit > 0 && !(scratch && scratch_bytes >= need && (reinterpret_cast<uintptr_t>(scratch) & 15) == 0)) nsplit = 0;
    const int nt = (Tk + 63) / 64;
    const AttnPlan plan = attention_plan(Bn, Tq, nt, heads, nsplit);
    // The unmeasured attempt saves a maximum per half tile and costs its check: from 20 tiles of plain keys on, always with prescaled ones.  (The line is as old
    // as a second attempt that spilled.  Now, us, measured / tried first: 2 x 4096 on 77 keys x 10 heads 9.66 / 9.79, 1 x 512 x 5 9.20 / 9.35, 4 x 400 x 20 13.2 / 12.7,
    // 8 x 512 x 10 13.8 / 13.1, 8 x 988 x 20 52.5 / 50.2, 8 x 1100 x 20 66.8 / 62.9, 4 x 1216 x 10 26.6 / 25.1.)
    const bool tries = k_prescaled || nt >= 20;
    SD_REQUIRE(plan.qb == 2 || (nsplit == 0 && tries), SD_EINVAL, "attention: 256 queries, but cut or measured");     // no such kernel, and scratch memory for 128
    if (nsplit > arrived_n) arrived = nullptr;   // not enough counters: the halves are merged by the second kernel
    *cut_tiles = arrived ? 0 : nsplit;
    // Read-ahead in the room that three workgroups to a CU leave: 8 MB and 2 MB per key tile, which the launch is long
    // enough for.  (With 1 MB per key tile the queue falls behind at 32 x 32 tokens: 2540 us per stack for 2500, 2658 without any.)
    // Workgroups of two groups have a CU each; what reads ahead runs beside them and behind.  (256 threads to each of the 448; ten blocks, with none of them / 128 / 256 /
    // 448 / 768 / 1024: 1 x 988 x 1280 + 16 1628 1563 1567 1492 1490 1487, 1 x 620 x 1280 + 64 1748 1699 1725 1598 1599 1598.)
    const int grid = attention_grid(plan.nfull, nsplit);
    const ReadRanges ra = ahead && k_prescaled ? ahead->take((8ull + 2 * nt) << 20, plan.gr == 1 ? 3l * device_cus() - grid : 7l * device_cus() / 4, 16) : ReadRanges{};
    if (SD_DRY_RUN("attention%s%s%s%s%s; ", k_prescaled ? " prescaled" : "", tries ? " try" : "", nsplit > 0 ? (arrived ? " cut" : " cut merge") : "", dry_ranges(ra), dry_tiles(64 * plan.qb, plan.gr))) return SD_OK;
    auto go = [&](auto kernel, const auto& ranges) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(grid + (ra.wgs + plan.gr - 1) / plan.gr)), dim3(256 * plan.gr), 0, stream, q, ldq, k, ldk, vt, ldvt, out, ldo, Tq, Tk, Tkp, heads,
                           plan.qtiles, c, plan.nfull, nsplit, static_cast<float*>(scratch), arrived, ranges);
    };
    auto kind = [&](auto qb, auto gr) {
        constexpr int QB = decltype(qb)::value, GR = decltype(gr)::value;
        if (k_prescaled && ra.wgs) go(attention_kernel<QB, GR, true, true, true>, ra);
        else if (k_prescaled) go(attention_kernel<QB, GR, true, true, false>, NoRanges{});
        else if (tries) go(attention_kernel<QB, GR, false, true, false>, NoRanges{});
        else if constexpr (QB == 2) go(attention_kernel<QB, GR, false, false, false>, NoRanges{});
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    if (plan.qb == 4 && plan.gr == 2) kind(I4{}, I2{});
    else if (plan.qb == 4) kind(I4{}, I1{});
    else if (plan.gr == 2) kind(I2{}, I2{});
    else kind(I2{}, I1{});
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

int launch_attention_merge(const void* scratch, uint16_t* out, int64_t ldo, int Bn, int Tq, int heads, bool k_prescaled, int cut_tiles,
                           hipStream_t stream) {
    if (cut_tiles <= 0 || SD_DRY_RUN("merge; ")) return SD_OK;
    // the halves' maxima are in score units, or already in exponent units when the keys were prescaled
    const float c = k_prescaled ? 1.0f : 0.125f * 1.44269504088896340736f;
    const AttnPlan p = attention_plan(Bn, Tq, 0, heads, cut_tiles);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)cut_tiles), dim3(256 * p.gr), 0, stream, static_cast<const float*>(scratch), out, ldo, Tq, heads, p.qtiles, p.nfull, c);
    };
    if (p.gr == 2) go(attention_merge_kernel<2, 2>);
    else go(attention_merge_kernel<2, 1>);
    SD_HIP_CHECK(hipGetLastError());
    return SD_OK;
}

}  // namespace sd
