// bdlm_mix.hip -- gfx950 kernels for a step or commit with the convolution part of the
// boundary state (App. C) on blocks of up to 256 tokens: the mixer's width-4 depthwise
// convolution with SiLU on x, B and C, forward continued from the cached rows and reverse
// zero-padded past the block (Sec. 4), then Eq. partial-reverse on the convolved inputs.
//
// With subscripts f and r for the forward and reverse convolutions,
//   y[t,:] = 2^{cs_t} (Cf_t . s^T)
//          + sum_{j<=t} Gf[t,j] 2^{cs_t - cs_j} dt_j xf[j,:] + D xf[t,:]
//          + sum_{j>=t} Gr[t,j] 2^{ex_j - ex_t} dt_j xr[j,:] + D_rev xr[t,:]
//   Gf[t,j] = Cf_t . Bf_j,  Gr[t,j] = Cr_t . Br_j
//   s_new  = 2^{cs_{L-1}} s + sum_j 2^{cs_{L-1} - cs_j} dt_j xf[j,:] (outer) Bf_j
//
// Everything here is fp32 and the matrix unit's fp32 rate is a sixteenth of its bf16 rate, so
// three things decide the time.
//   G does not depend on the head: a first kernel convolves B and C once per (batch row,
//   group) and forms the Gram tiles (fp32 MFMA), so that a head's workgroup reads them from
//   L2 instead of convolving B and C and forming all of G again.
//   fp32 products run as bf16 ones: an operand is split into three bf16 terms, v = h + m + l,
//   exact to 2^-26, and a product takes the six terms hh, hm, mh, hl, lh, mm (the three left
//   out are below 2^-25 of it, half an ulp of an fp32 product).  Six 32-deep bf16 MFMAs
//   against eight 4-deep fp32 ones per 32 indices: 96 against 256 matrix cycles per tile.
//   The decays are not applied to G: 2^{cs_t - cs_j} factors into a weight of the source token
//   relative to the end of its pair of tiles (folded into x before it is split), one scalar
//   per pair of tiles (the accumulator is scaled as it passes from one pair to the next, as
//   in Horner's rule) and a weight of the row (applied once, to the result).  So G is masked
//   and split once per group by the first kernel, and the head kernel's inner loop is loads
//   and MFMAs.  A pair of tiles over which the state decays below 2^-60 takes a path of its
//   own (pair_slow); the source weights stay at or above 2^-60, so no factor overflows.
//
// Measured (26 heads, dstate 128, block 256, batch 16, bf16 inputs, traced): a step 19 + 60 us,
// a commit 19 + 83 us, against 28 us for the convolution into an fp32 workspace and 85 + 82 us
// for the sequence kernels' forward and reverse launches on it (fp32 MFMA), which blocks of
// more than 256 tokens still take.  At 32 heads and 64 tokens, step and commit with the
// normalisation between them: 68 us against 144.  What bounds the head kernel, step | commit: waves
// wait for memory, LDS and barriers 51 | 60 % of their time and for an issue slot 28 | 23 %, with
// the vector ALU busy in 33 | 28 % of the cycles (half of it the convolution and its split) and the
// matrix unit in 22 | 21 %; the commit holds outputs and states side by side in 128 registers and
// spills 39 (75 in fp32; 160 and 176 bytes a lane), the step 56 to 68 bytes a lane.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bdlm.h"
#include "bdlm_device.h"
#include "bdlm_images.h"
#include "bdlm_launch.h"

namespace bdlm {
namespace {

struct MixArgs {
    const void *x, *dt, *Bm, *Cm;  // before the convolution
    const float *A, *D, *D_rev;
    const float *w, *bias;         // [channels][4] (w[c][3] on the current token), [channels]
    float *cache;                  // [nslots][3][channels] input rows; a commit replaces them
    float *pool;                   // cached states; a commit updates them in place
    float *y;                      // outputs, or nullptr (a commit without them)
    uint4 *gram;                   // per (row, group): nt (np + 1) pairs of Gram tiles of 3 x 64
    uint2 *c3, *b3;                // per (row, group): Cf [nt][NP / 32][3] and Bf^T [N / 16][np][3]
                                   // MFMA operands of 64 lanes x 16 bytes (NP: N, at least 32)
    int64_t xs_b, xs_t, xs_h, dts_b, dts_t, bcs_b, bcs_t, bcs_g;
    int32_t L, nt, np;             // tokens; 16-token tiles; pairs of them
    int32_t batch, nheads, ngroups, heads_per_group, channels;
    int32_t commit, xcd_remap, use_slots;
    int32_t slots[BDLM_MAX_SLOT_ROWS];
};

typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const f32x4 g_f4;
typedef __attribute__((address_space(1))) const uint16_t g_u16;
typedef __attribute__((address_space(1))) const float g_f;

__device__ __forceinline__ float ex2(float v) { return __builtin_amdgcn_exp2f(v); }

// v / (1 + e^-v) = q + t r: a quotient q by the hardware reciprocal r and its remainder t = (v - q)
// - q e^-v, which does without the rounding of 1 + e^-v (v - q is exact for v >= 0, where the
// function is large).  Past 88 either way q is v or 0 by itself (infinities: +inf and NaN, as a
// division gives), and the remainder, in which infinities would meet, is left out.
struct Silu {
    float q, r, t;
};
__device__ __forceinline__ Silu silu(float v) {
    const float e = ex2(v * -kLog2e);
    const float r = __builtin_amdgcn_rcpf(1.f + e);
    const float q = v * r;
    // (formed, then selected: as one expression it compiles to a branch)
    const float t = fmaf(-q, e, v - q);
    return Silu{q, r, fabsf(v) < 88.f ? t : 0.f};
}

// Four floats as three bf16 quads (rounded, not cut: the terms alternate in sign, and the
// products that mma6 leaves out are a sixteenth of what they would be).
struct T3 {
    uint2 t[3];
};
__device__ __forceinline__ T3 split3(f32x4 v) {
    s16x4 h, m, l;
    split4x3(v, h, m, l);
    return T3{{as_u2(h), as_u2(m), as_u2(l)}};
}
__device__ __forceinline__ f32x4 quad_val(uint2 v) {
    return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                 __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
}
__device__ __forceinline__ f32x4 join3(uint2 h, uint2 m, uint2 l) {
    return quad_val(h) + (quad_val(m) + quad_val(l));
}
__device__ __forceinline__ f32x4 mma_pair(uint4 a, uint4 b, f32x4 c) {
    return mma_k32(as_s16x4(uint2{a.x, a.y}), as_s16x4(uint2{a.z, a.w}), as_s16x4(uint2{b.x, b.y}),
                   as_s16x4(uint2{b.z, b.w}), c);
}
// a b over 32 contraction indices, both operands in three terms (smallest products first).  The
// sum starts from zero and is added to an accumulator once: six products added to it one by one
// would each round at its size.
__device__ __forceinline__ f32x4 mma6(const uint4 (&a)[3], const uint4 (&b)[3]) {
    f32x4 c = mma_pair(a[1], b[1], f32x4{0.f, 0.f, 0.f, 0.f});
    c = mma_pair(a[2], b[0], c);
    c = mma_pair(a[0], b[2], c);
    c = mma_pair(a[1], b[0], c);
    c = mma_pair(a[0], b[1], c);
    return mma_pair(a[0], b[0], c);
}
__device__ __forceinline__ f32x4 mma_q32(f32x4 a, f32x4 b, f32x4 c) {
#pragma unroll
    for (int r = 0; r < 4; ++r) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b[r], c, 0, 0, 0);
    return c;
}

// Rows through a buffer resource at the channels' first element: a row outside the block gets
// an offset past the resource's range and loads zeros (L rows of at most 2^31 bytes: mix_fits).
constexpr uint32_t kOOB = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), static_cast<short>(0), 0x7fffffff,
                                             0x00020000);
}

// The convolution of four channels over four tokens t0 .. t0 + 3: rows t0-3 .. t0+3 (forward)
// or t0 .. t0+6 (reverse) of the input; before the block the cached rows, past it zeros.
// BF16: rows are kept as they were loaded, two channels to a register.
template <bool BF16, bool REV>
struct ConvTask {
    f32x4 w[4], b;       // per channel: its four weights; biases
    u32x4 u[7];          // bf16: two words used
    f32x4 old[3];        // the cached rows, where t0 == 0 (forward)
    bool first;
    __device__ __forceinline__ void weights(const MixArgs &a, int c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = *(const g_f4 *)(a.w + 4 * static_cast<int64_t>(c + e));
        b = *(const g_f4 *)(a.bias + c);
    }
    // src: the row's block; off: byte offset of these channels' elements of token 0 in it; rs:
    // bytes between tokens; crow: the channels' cached rows (stride a.channels)
    __device__ __forceinline__ void load(const void *src, uint32_t off, uint32_t rs, const float *crow,
                                         const MixArgs &a, int t0) {
        const __amdgpu_buffer_rsrc_t r = rsrc(src);
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int t = REV ? t0 + i : t0 - 3 + i;
            const uint32_t o = static_cast<uint32_t>(t) < static_cast<uint32_t>(a.L) ? off + t * rs : kOOB;
            if constexpr (BF16) {
                const v2u v = __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0);
                u[i] = u32x4{v.x, v.y, 0u, 0u};
            } else {
                u[i] = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
            }
        }
        if constexpr (!REV) {
            // unconditional, as every load here (a zero chunk where a row is not wanted)
            first = t0 == 0;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                old[i] = *(first ? (const g_f4 *)(crow + static_cast<int64_t>(i) * a.channels) : (const g_f4 *)(&kZeroChunk));
        }
    }
    // channel e at the four tokens (past the block: some finite value, which meets source
    // weights of zero or rows that are not stored)
    // (skip, unless null: the values times D, before the values' rounding)
    __device__ __forceinline__ f32x4 out(int e, float D = 0.f, f32x4 *skip = nullptr) const {
        float v[7];
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            if constexpr (BF16) {
                const uint32_t x = e < 2 ? u[i].x : u[i].y;
                v[i] = __uint_as_float(e & 1 ? x & 0xffff0000u : x << 16);
            } else {
                v[i] = __uint_as_float(u[i][e]);
            }
            if constexpr (!REV)
                if (i < 3) v[i] += old[i][e];          // one of the two is zero
        }
        f32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float s = b[e];
#pragma unroll
            for (int k = 0; k < 4; ++k) s += w[e][k] * (REV ? v[i + 3 - k] : v[i + k]);
            const Silu u = silu(s);
            o[i] = fmaf(u.t, u.r, u.q);
            if (skip) (*skip)[i] = fmaf(D, u.q, D * (u.t * u.r));
        }
        return o;
    }
};

// ------------------------------------------------------------------ the Gram kernel
// Workgroups per (row, group): blocks of 64 tokens t by 64 tokens j, the forward ones on and
// below the diagonal and the reverse ones on and above it.  Wave w forms the tiles (mt, 2 jp)
// and (mt, 2 jp + 1) of row tile mt = w % 4, pair w / 4 of its block, masks them (j <= t
// forward, j >= t reverse), splits them and stores them as the A operand of the head kernel:
// lane (grp, col) of term z holds G[16 mt + col][32 jp + 4 grp .. +3] and the same 16 tokens
// on.  Forward pairs (jp <= mt / 2) at mt (np + 1) + jp, reverse ones (jp >= mt / 2) one
// further.  The forward workgroups of the diagonal also store Cf and, for a commit, Bf^T in
// three terms.
// (64 x 64 blocks: 320 workgroups at batch 16 and 256 tokens.  Every workgroup convolves its
// 128 token rows again, 2.5 times the work of convolving each row once, but in one launch.)
template <int NS, bool BF16>
__global__ void __launch_bounds__(512) bdlm_mix_gram_kernel(const MixArgs a) {
    constexpr int QN = NS / 16, CQ = NS / 4, ES = BF16 ? 2 : 4, NP = NS < 32 ? 32 : NS;
    constexpr int TASKS = 2 * CQ * 16;                 // (matrix, token quad, channel quad)
    constexpr int PT = TASKS >= 512 ? TASKS / 512 : 1;
    __shared__ __align__(16) f32x4 sI[2][4 * QN * 64]; // operand images of C and B
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int nb = (a.L + 63) / 64;
    const bool want_y = a.y != nullptr;
    int u = blockIdx.x;
    int ji = 0;
    if (want_y) {
        ji = u % (nb + 1);
        u /= nb + 1;
    }
    const int mi = u % nb;
    u /= nb;
    const int g = u % a.ngroups, b = u / a.ngroups;
    if (!want_y) ji = mi;              // a commit without outputs: the diagonal's, for Bf^T
    const bool rev = ji > mi;
    if (rev) --ji;
    const bool diag = mi == ji && !rev;
    const int bg = b * a.ngroups + g;
    const int64_t slot = a.use_slots ? a.slots[b] : b;
    const int HP = a.nheads * kP, GN = a.ngroups * NS;
    const float *crow = a.cache + slot * 3 * static_cast<int64_t>(a.channels);

    auto convolve = [&](auto rev_tag) {
        constexpr bool REV = decltype(rev_tag)::value;
        ConvTask<BF16, REV> tk[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const int task = (tid + 512 * k) % TASKS, m = task / (CQ * 16), cq = task % CQ;
            const int t0 = 64 * (m == 0 ? mi : ji) + 4 * ((task / CQ) & 15);
            const int c = HP + (m == 0 ? GN : 0) + g * NS + 4 * cq;
            // (one matrix per k where there are two: its base is uniform)
            const char *src = static_cast<const char *>((PT == 2 ? k == 0 : m == 0) ? a.Cm : a.Bm) +
                              (b * a.bcs_b + g * a.bcs_g) * ES;
            if constexpr (PT == 2) {
                tk[k].load(src, 4 * cq * ES, static_cast<uint32_t>(a.bcs_t) * ES, crow + c, a, t0);
            } else {
                const char *bB = static_cast<const char *>(a.Bm) + (b * a.bcs_b + g * a.bcs_g) * ES;
                const char *bC = static_cast<const char *>(a.Cm) + (b * a.bcs_b + g * a.bcs_g) * ES;
                if (m == 0) tk[k].load(bC, 4 * cq * ES, static_cast<uint32_t>(a.bcs_t) * ES, crow + c, a, t0);
                else tk[k].load(bB, 4 * cq * ES, static_cast<uint32_t>(a.bcs_t) * ES, crow + c, a, t0);
            }
            tk[k].weights(a, c);
        }
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const int task = tid + 512 * k, m = task / (CQ * 16), cq = task % CQ;
            if (TASKS < 512 && task >= TASKS) break;
            const int tl = 4 * ((task / CQ) & 15), t0 = 64 * (m == 0 ? mi : ji) + tl;
            f32x4 ch[4], v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) ch[e] = tk[k].out(e);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = f32x4{ch[0][i], ch[1][i], ch[2][i], ch[3][i]};
                sI[m][((tl >> 4) * QN + (cq >> 2)) * 64 + (cq & 3) * 16 + (((tl & 15) + i) ^ (cq & 15))] = v[i];
            }
            if constexpr (!REV) {
                if (diag && m == 0 && want_y && t0 < 16 * a.nt) {
                    // row tile t0 / 16, 32 channels cq / 8: lane (grp, col) holds channels 8 grp ..
                    // +7 of token col
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const T3 s = split3(v[i]);
                        uint2 *dst = a.c3 + ((static_cast<int64_t>(bg) * a.nt + (t0 >> 4)) * (NP / 32) + (cq >> 3)) * 384 +
                                     2 * (16 * ((cq >> 1) & 3) + (t0 & 15) + i) + (cq & 1);
#pragma unroll
                        for (int z = 0; z < 3; ++z) dst[128 * z] = s.t[z];
                    }
                }
                if (diag && m == 1 && a.commit && t0 < 32 * a.np) {
                    // dstate tile cq / 4, token pair-tile t0 / 32: lane (grp, col) holds tokens 4 grp
                    // .. +3 and the four 16 further on of channel 16 (cq / 4) + col
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const T3 s = split3(ch[e]);
                        uint2 *dst = a.b3 + ((static_cast<int64_t>(bg) * QN + (cq >> 2)) * a.np + (t0 >> 5)) * 384 +
                                     2 * (16 * ((t0 >> 2) & 3) + 4 * (cq & 3) + e) + ((t0 >> 4) & 1);
#pragma unroll
                        for (int z = 0; z < 3; ++z) dst[128 * z] = s.t[z];
                    }
                }
            }
        }
    };
    if (rev) convolve(std::true_type{});
    else convolve(std::false_type{});
    if (!want_y) return;
    __syncthreads();
    const int mt = 4 * mi + (wave & 3), jp = 2 * ji + (wave >> 2);
    if (mt >= a.nt || jp >= a.np || (rev ? jp < (mt >> 1) : jp > (mt >> 1))) return;
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int q = 0; q < QN; ++q) {
        const f32x4 c = sI[0][img_idx<QN, true>(wave & 3, q, grp, col)];
#pragma unroll
        for (int d = 0; d < 2; ++d)
            acc[d] = mma_q32(sI[1][img_idx<QN, true>(2 * (wave >> 2) + d, q, grp, col)], c, acc[d]);
    }
    T3 s[2];
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const int t = 16 * mt + col, j = 32 * jp + 16 * d + 4 * grp;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (rev ? j + r < t : j + r > t) acc[d][r] = 0.f;
        s[d] = split3(acc[d]);
    }
    uint4 *dst = a.gram + (static_cast<int64_t>(bg) * a.nt * (a.np + 1) + mt * (a.np + 1) + jp + (rev ? 1 : 0)) * 192 + lane;
#pragma unroll
    for (int z = 0; z < 3; ++z) dst[64 * z] = uint4{s[0].t[z].x, s[0].t[z].y, s[1].t[z].x, s[1].t[z].y};
}

// ------------------------------------------------------------------ the head kernel
// One workgroup of NW waves per (row, head); wave w owns the output rows of one tile of each
// block of NW tiles (MR blocks: L <= 16 NW MR).  Source tokens are convolved, weighted and
// staged a block (TB = 16 NW tokens) and a direction at a time, in one LDS image of 48 KB at
// most, so that two workgroups share a CU and one convolves while the other multiplies.
template <int NW> struct XImg {
    static constexpr int TB = 16 * NW, CH = TB / 8;    // tokens; 16-byte chunks per column
    static constexpr int PLANE = kP * CH;              // chunks per term
    // Chunk c (lane group c % 4 of token pair-tile c / 4: tokens 32 (c/4) + 4 (c%4) .. +3 and
    // the four 16 further on) of column p.  XOR-permuted so that the reads (16 columns, one
    // chunk) and the writes (16 column quads, one chunk half) meet distinct banks.
    static __device__ __forceinline__ int at(int p, int c) {
        if constexpr (CH >= 16) return p * CH + (c ^ (p & 15) ^ (p >> 4));
        else return p * CH + (c ^ ((p >> 1) & 7) ^ (p >> 5));
    }
};
constexpr float kLeast = -60.f;                        // log2 of the least source weight

template <int NW, int MR, int NS, bool BF16, bool COMMIT>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 8 ? 4 : 2)))
bdlm_mix_kernel(const MixArgs a) {
    using XI = XImg<NW>;
    constexpr int NT = 64 * NW, TB = XI::TB;
    constexpr int NTOK = TB * MR, TPL = NTOK / 64, NPAIR = NTOK / 32;
    constexpr int QN = NS / 16;
    constexpr int NP = NS < 32 ? 32 : NS;              // dstate padded to one 32-deep operand
    constexpr int SCH = NP / 8;                        // chunks per column of the state image
    constexpr int XB = 3 * XI::PLANE, SB = 3 * kP * SCH;
    static_assert(XI::TB * 4 == 64 * NW, "one convolution task per thread");
    __shared__ __align__(16) uint4 sX[XB > SB ? XB : SB];
    __shared__ __align__(16) float sEc[NTOK];               // 2^{cs_t}
    // pair_slow: log2 decays from the own pair's far end, in two floats (forward, reverse)
    __shared__ __align__(16) float2 sCs[NTOK], sEx[NTOK];
    __shared__ __align__(16) float sWf[NTOK], sWr[NTOK];    // source weights (times dt)
    __shared__ __align__(16) float sRf[NTOK], sRr[NTOK];    // row weights, from the own pair
    __shared__ __align__(16) float sRx[MR > 1 ? NTOK : 4];  // row weights, from the other block
    __shared__ float sQ[NPAIR];                             // decay of a pair of tiles
    __shared__ float2 sD[NPAIR];                            // and its log2, in two floats

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    int un = blockIdx.x;
    if (a.xcd_remap) un = (un & 7) * (static_cast<int>(gridDim.x) >> 3) + (un >> 3);
    const int b = un / a.nheads, h = un - b * a.nheads, g = h / a.heads_per_group;
    const int64_t slot = a.use_slots ? a.slots[b] : b;
    const int L = a.L, nt = a.nt, np = a.np;
    const int bg = b * a.ngroups + g;
    const bool want_y = a.y != nullptr;
    float *hs = a.pool + (slot * a.nheads + h) * (kP * NS);
    // waves w and w + 4 share a SIMD: row tiles w and 7 - w, so that every SIMD has the same
    // number of tiles in the triangular blocks
    const int ml = NW == 8 ? (wave < 4 ? wave : 11 - wave) : wave;

    // this thread's convolution task: channels h * 64 + 4 cq .. +3, tokens 4 tq .. +3 of a block
    const int cq = tid & 15, tq = tid >> 4;
    constexpr int ES = BF16 ? 2 : 4;
    const char *xg = static_cast<const char *>(a.x) + (b * a.xs_b + h * a.xs_h) * ES;
    float *crow = a.cache + slot * 3 * static_cast<int64_t>(a.channels) + h * kP + 4 * cq;
    const float Df = a.D[h], Dr = a.D_rev[h];
    const uint32_t ytokB = static_cast<uint32_t>(a.nheads) * kP * 4;
    float *ybase = a.y + (static_cast<int64_t>(b) * L * a.nheads + h) * kP;

    // ---- decay sums and per-token factors (wave 0, TPL tokens per lane).  The sums run in
    // double: over 256 tokens a float's ulp of cs would show in every weight.
    if (wave == 0) {
        const char *dtg = static_cast<const char *>(a.dt) + (b * a.dts_b + h) * (BF16 ? 2 : 4);
        float dtv[TPL];
        double cs[TPL], ex[TPL];
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            const int t = TPL * lane + i;
            const bool ok = t < L;
            if constexpr (BF16)
                dtv[i] = __uint_as_float(static_cast<uint32_t>(*(ok ? (const g_u16 *)(dtg + t * a.dts_t * 2)
                                                                     : (const g_u16 *)(&kZeroChunk)))
                                         << 16);
            else
                dtv[i] = *(ok ? (const g_f *)(dtg + t * a.dts_t * 4) : (const g_f *)(&kZeroChunk));
        }
        const double A2 = a.A[h] * 1.4426950408889634;
        double run = 0.;
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            run += dtv[i] * A2;
            cs[i] = run;
        }
        const double excl = wave_inclusive_sum_d(run) - run;
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            ex[i] = i == 0 ? excl : cs[i - 1];
            cs[i] += excl;
        }
        constexpr int LPP = 32 / TPL;                  // lanes per pair of tiles
        auto two = [](double v) {
            const float hi = static_cast<float>(v);
            return float2{hi, static_cast<float>(v - hi)};
        };
        const int p = lane / LPP;
        const double E = __shfl(cs[TPL - 1], LPP * p + LPP - 1, 64);   // the pair's end
        const double S = __shfl(ex[0], LPP * p, 64);                   // and its start
        const double X = MR > 1 ? __shfl(cs[TPL - 1], 31, 64) : 0.;    // the first block's end
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            const int t = TPL * lane + i;
            sCs[t] = two(cs[i] - E);
            sEx[t] = two(S - ex[i]);
            sEc[t] = ex2(static_cast<float>(cs[i]));
            sWf[t] = ex2(fmaxf(static_cast<float>(E - cs[i]), kLeast)) * dtv[i];
            sWr[t] = ex2(fmaxf(static_cast<float>(ex[i] - S), kLeast)) * dtv[i];
            sRf[t] = ex2(static_cast<float>(cs[i] - E));
            sRr[t] = ex2(static_cast<float>(S - ex[i]));
            if constexpr (MR > 1) sRx[t] = ex2(static_cast<float>(t < TB ? X - ex[i] : cs[i] - X));
        }
        if (lane % LPP == LPP - 1) {
            sD[p] = two(E - S);
            sQ[p] = ex2(static_cast<float>(E - S));
        }
    }

    f32x4 Y[MR][4];
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) Y[m][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint2 *sX2 = reinterpret_cast<uint2 *>(sX);
    const uint4 *gram = a.gram + static_cast<int64_t>(bg) * nt * (np + 1) * 192 + lane;
    const uint4 *c3 = reinterpret_cast<const uint4 *>(a.c3) + static_cast<int64_t>(bg) * nt * (NP / 32) * 192 + lane;
    const uint4 *b3 = reinterpret_cast<const uint4 *>(a.b3) + static_cast<int64_t>(bg) * QN * np * 192 + lane;
    // The heads of a group run side by side and need the same tiles at the same time, each for
    // the first time: they would all wait for memory at every tile.  So the group's workgroups
    // first request a share each of the lines, one word a line, into their L2.
    uint32_t warm = 0u;
    {
        // 128-byte lines (a commit without outputs reads Bf^T alone)
        const int nl = want_y ? nt * (np + 1) * 24 : 0, ncl = want_y ? nt * (NP / 32) * 24 : 0, nbl = COMMIT ? QN * np * 24 : 0;
        for (int i = (h - g * a.heads_per_group) * NT + tid; i < nl + ncl + nbl; i += a.heads_per_group * NT) {
            const uint4 *src = i < nl ? gram - lane + i * 8 : (i < nl + ncl ? c3 - lane + (i - nl) * 8 : b3 - lane + (i - nl - ncl) * 8);
            warm ^= src->x;
        }
    }
    if (want_y) {
        // ---- prefix term 2^{cs_t} (Cf_t . s^T), before the x image takes the LDS: the state in
        // three terms, columns' chunks XOR-permuted like the x image's
        auto s_at = [&](int p, int c) {
            return p * SCH + (c ^ (SCH >= 16 ? (p & 15) : (SCH == 8 ? (p >> 1) & 7 : (p >> 2) & 3)));
        };
        constexpr int SQ = kP * NP / 4;                // quads of the (padded) state
#pragma unroll
        for (int i = tid; i < SQ; i += NT) {
            const int p = i & 63, n4 = i >> 6;
            const f32x4 v = 4 * n4 < NS ? *reinterpret_cast<const f32x4 *>(hs + static_cast<int64_t>(i) * 4)
                                        : f32x4{0.f, 0.f, 0.f, 0.f};
            const T3 s = split3(v);
            const int at = 2 * s_at(p, n4 >> 1) + (n4 & 1);
#pragma unroll
            for (int z = 0; z < 3; ++z) sX2[2 * z * kP * SCH + at] = s.t[z];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NP / 32; ++k) {
            uint4 cf[MR][3];
#pragma unroll
            for (int m = 0; m < MR; ++m)
#pragma unroll
                for (int z = 0; z < 3; ++z) {
                    const int mt = min(NW * m + ml, nt - 1);
                    const bool ok = 32 * k + 8 * grp < NS;
                    const g_u4 *src = ok ? gchunk(c3 + ((mt * (NP / 32) + k) * 3 + z) * 64) : gzero();
                    cf[m][z] = __builtin_bit_cast(uint4, *src);
                }
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) {
                uint4 sq[3];
#pragma unroll
                for (int z = 0; z < 3; ++z) sq[z] = sX[z * kP * SCH + s_at(16 * ct + col, 4 * k + grp)];
#pragma unroll
                for (int m = 0; m < MR; ++m) Y[m][ct] += mma6(cf[m], sq);
            }
        }
#pragma unroll
        for (int m = 0; m < MR; ++m) {
            const f32x4 ec = *reinterpret_cast<const f32x4 *>(&sEc[16 * (NW * m + ml) + 4 * grp]);
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) Y[m][ct] *= ec;
        }
    }
    // commit: this wave's tiles of the state, dstate tiles q0 .. q0 + QW - 1 by column tiles c0 ..
    // c0 + CW - 1 (whole rows of tiles where there are enough: Bf^T comes from memory, x from LDS)
    constexpr int QW = QN >= NW ? QN / NW : 1, CW = QN >= NW ? 4 : (4 * QN >= NW ? 4 * QN / NW : 1);
    const int q0 = QN >= NW ? wave * QW : wave % QN, c0 = QN >= NW ? 0 : wave / QN * CW;
    const bool owns = c0 < 4;
    f32x4 acc[COMMIT ? QW : 1][COMMIT ? CW : 1];
    auto state_at = [&](int k, int c) { return hs + ((4 * (q0 + k) + grp) * kP + 16 * (c0 + c) + col) * 4; };
    if constexpr (COMMIT) {
        if (owns) {
#pragma unroll
            for (int k = 0; k < QW; ++k)
#pragma unroll
                for (int c = 0; c < CW; ++c) acc[k][c] = *reinterpret_cast<const f32x4 *>(state_at(k, c));
        }
    }
    asm volatile("" ::"v"(warm));
    __syncthreads();   // the decay factors are there; the state image is overwritten
    const int wc = 4 * (tq >> 3) + (tq & 3), whalf = (tq >> 2) & 1;   // where the task's tokens go

    const int nblk = MR == 1 ? 1 : (L + TB - 1) / TB;
    auto stage = [&](auto rev_tag, int sb) {
        constexpr bool rev = decltype(rev_tag)::value;
        // ---- convolve this stage's tokens into the image (rows and weights are loaded here:
        // held over the products they would not fit in the registers of four waves per SIMD,
        // and the CU's other workgroup works meanwhile)
        {
            const int t0 = TB * sb + 4 * tq;
            ConvTask<BF16, rev> tk;
            tk.load(xg, 4 * cq * ES, static_cast<uint32_t>(a.xs_t) * ES, crow, a, t0);
            tk.weights(a, h * kP + 4 * cq);
            // the skip terms go straight to y, the reverse one added onto the forward one by the
            // thread that wrote it (the rows' waves add the rest in the end)
            const __amdgpu_buffer_rsrc_t rY = rsrc(ybase);
            uint32_t yo[4];
            f32x4 sk[4], yv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                yo[i] = t0 + i < L ? static_cast<uint32_t>(t0 + i) * ytokB + 16 * cq : kOOB;
                if constexpr (rev) yv[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rY, yo[i], 0, 0));
            }
            const f32x4 wt = *reinterpret_cast<const f32x4 *>((rev ? sWr : sWf) + t0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f32x4 o = rev ? tk.out(e) : tk.out(e, Df, &sk[e]);
                if constexpr (rev) sk[e] = Dr * o;
                const T3 s = split3(o * wt);
                const int at = 2 * XI::at(4 * cq + e, wc) + whalf;
#pragma unroll
                for (int z = 0; z < 3; ++z) sX2[2 * z * XI::PLANE + at] = s.t[z];
            }
            if (want_y) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    f32x4 v = {sk[0][i], sk[1][i], sk[2][i], sk[3][i]};
                    if constexpr (rev) v += yv[i];
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rY, yo[i], 0, 0);
                }
            }
        }
        __syncthreads();
        if (want_y) {
            // ---- the block's pairs of source tiles into this wave's rows, towards the row: each
            // step scales what is there by the decay of the pair passed and adds the pair
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                const int mt = NW * m + ml;
                if (mt >= nt || (rev ? m > sb : m < sb)) continue;
                const int first = NW / 2 * sb, last = min(first + NW / 2, np) - 1;
                const int own = mt >> 1;               // the pair that holds the row itself
                const bool slow = m == sb && sQ[own] < 8.6736174e-19f;   // 2^-60
                // forward pairs first .. (m == sb ? own : last), reverse ones last down to (own or first)
                int jp = rev ? last : first;
                const int end = m == sb ? own : (rev ? first : last), dj = rev ? -1 : 1;
                const int n = (end - jp) * dj + (slow ? 0 : 1);
                f32x4 T[4];
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) T[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
                const uint4 *gp = gram + (mt * (np + 1) + (rev ? 1 : 0)) * 192;
                uint4 M[3];
#pragma unroll
                for (int z = 0; z < 3; ++z) M[z] = gp[jp * 192 + 64 * z];
#pragma unroll 1
                for (int i = 0; i < n; ++i, jp += dj) {
                    uint4 N[3];
                    const int nx = i + 1 < n ? jp + dj : jp;
#pragma unroll
                    for (int z = 0; z < 3; ++z) N[z] = gp[nx * 192 + 64 * z];
                    const float q = sQ[jp];
#pragma unroll
                    for (int ct = 0; ct < 4; ++ct) {
                        uint4 xq[3];
#pragma unroll
                        for (int z = 0; z < 3; ++z)
                            xq[z] = sX[z * XI::PLANE + XI::at(16 * ct + col, 4 * (jp - first) + grp)];
                        T[ct] = T[ct] * q + mma6(M, xq);
                    }
#pragma unroll
                    for (int z = 0; z < 3; ++z) M[z] = N[z];
                }
                // the row weights: from the own pair's far end, or the block's end
                f32x4 f;
                if (MR > 1 && m != sb) f = *reinterpret_cast<const f32x4 *>(&sRx[16 * mt + 4 * grp]);
                else if (!slow) f = *reinterpret_cast<const f32x4 *>((rev ? sRr : sRf) + 16 * mt + 4 * grp);
                else {
                    int g4 = 4 * grp;
                    asm volatile("" : "+v"(g4));
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int t = 16 * mt + g4 + r;
                        const float2 c = (rev ? sEx : sCs)[t], D = sD[own];
                        f[r] = ex2((c.x + D.x) + (c.y + D.y));
                    }
                }
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) Y[m][ct] += f * T[ct];
                if (slow) {
                    // ---- pair_slow: the own pair's decays element by element, in G (undoing the
                    // source weight, which is the decay to the pair's end or 2^-60)
                    int grp_ = grp, col_ = col;        // nothing of this path is formed ahead of it
                    asm volatile("" : "+v"(grp_), "+v"(col_));
                    const uint4 g0 = gp[own * 192], g1 = gp[own * 192 + 64], g2 = gp[own * 192 + 128];
                    const int t = 16 * mt + col_;
                    const float2 ct2 = (rev ? sEx : sCs)[t];
                    T3 s[2];
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        f32x4 v = d == 0 ? join3(uint2{g0.x, g0.y}, uint2{g1.x, g1.y}, uint2{g2.x, g2.y})
                                         : join3(uint2{g0.z, g0.w}, uint2{g1.z, g1.w}, uint2{g2.z, g2.w});
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int j = 32 * own + 16 * d + 4 * grp_ + r;
                            const float2 cj = (rev ? sEx : sCs)[j];
                            const bool in = rev ? j >= t : j <= t;
                            // the decay from j to t less the weight that x_j holds
                            const float e = fminf(ct2.x, (ct2.x - cj.x) + (ct2.y - cj.y) - kLeast);
                            v[r] = in ? v[r] * ex2(e) : 0.f;
                        }
                        s[d] = split3(v);
                    }
#pragma unroll
                    for (int z = 0; z < 3; ++z) M[z] = uint4{s[0].t[z].x, s[0].t[z].y, s[1].t[z].x, s[1].t[z].y};
#pragma unroll
                    for (int ct = 0; ct < 4; ++ct) {
                        uint4 xq[3];
#pragma unroll
                        for (int z = 0; z < 3; ++z)
                            xq[z] = sX[z * XI::PLANE + XI::at(16 * ct + col_, 4 * (own - first) + grp_)];
                        Y[m][ct] += mma6(M, xq);
                    }
                }
            }
        }
        if constexpr (COMMIT) {
            // ---- the block's tokens into the new state, pair by pair: Bf^T (from memory) against
            // the weighted x
            if constexpr (!rev) {
                const int p0 = NW / 2 * sb, p1 = min(p0 + NW / 2, np);
                // (an operand is requested while the one before it multiplies)
                auto load_b = [&](int k, int jp, uint4 (&v)[3]) {
#pragma unroll
                    for (int z = 0; z < 3; ++z) v[z] = b3[((q0 + k) * np + jp) * 192 + 64 * z];
                };
                if (owns) {
                    uint4 bc[3], bn[3];
                    load_b(0, p0, bc);
#pragma unroll 1
                    for (int jp = p0; jp < p1; ++jp) {
                        const float q = sQ[jp];
#pragma unroll
                        for (int k = 0; k < QW; ++k) {
                            load_b(k + 1 < QW ? k + 1 : 0, k + 1 < QW || jp + 1 == p1 ? jp : jp + 1, bn);
#pragma unroll
                            for (int c = 0; c < CW; ++c) {
                                uint4 xq[3];
#pragma unroll
                                for (int z = 0; z < 3; ++z)
                                    xq[z] = sX[z * XI::PLANE + XI::at(16 * (c0 + c) + col, 4 * (jp - p0) + grp)];
                                acc[k][c] = acc[k][c] * q + mma6(bc, xq);
                            }
#pragma unroll
                            for (int z = 0; z < 3; ++z) bc[z] = bn[z];
                        }
                    }
                }
            }
        }
        __syncthreads();   // the image is rewritten
    };
#pragma unroll 1
    for (int sb = 0; sb < nblk; ++sb) {
        stage(std::false_type{}, sb);
        if (want_y) stage(std::true_type{}, sb);
    }

    if (want_y) {
        const __amdgpu_buffer_rsrc_t rY = rsrc(ybase);
#pragma unroll
        for (int m = 0; m < MR; ++m) {
            const int t0 = 16 * (NW * m + ml) + 4 * grp;
            float v[4][4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t o = t0 + r < L ? static_cast<uint32_t>(t0 + r) * ytokB + 4 * col : kOOB;
#pragma unroll
                for (int ct = 0; ct < 4; ++ct)
                    v[r][ct] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rY, o, 64 * ct, 0));
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t o = t0 + r < L ? static_cast<uint32_t>(t0 + r) * ytokB + 4 * col : kOOB;
#pragma unroll
                for (int ct = 0; ct < 4; ++ct)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[r][ct] + Y[m][ct][r]), rY, o, 64 * ct, 0);
            }
        }
    }
    if constexpr (COMMIT) {
        // every read of the state and of this head's cached rows is behind a barrier
        if (owns) {
#pragma unroll
            for (int k = 0; k < QW; ++k)
#pragma unroll
                for (int c = 0; c < CW; ++c) *reinterpret_cast<f32x4 *>(state_at(k, c)) = acc[k][c];
        }
        // the cached input rows: the last three of (cached rows ++ block); x by its head's
        // workgroup, B and C (which only the Gram kernel reads) by the group's first one
        auto keep_rows = [&](const char *src, int64_t rs, float *row) {
            float r[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int64_t t = static_cast<int64_t>(L) - 3 + k;   // < 0: an older cached row
                if (t < 0) r[k] = row[(t + 3) * a.channels];
                else if constexpr (BF16)
                    r[k] = __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t *>(src)[t * rs]) << 16);
                else r[k] = reinterpret_cast<const float *>(src)[t * rs];
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) row[k * static_cast<int64_t>(a.channels)] = r[k];
        };
        float *rows = a.cache + slot * 3 * static_cast<int64_t>(a.channels);
        if (tid < kP)
            keep_rows(static_cast<const char *>(a.x) + (b * a.xs_b + h * a.xs_h + tid) * ES, a.xs_t, rows + h * kP + tid);
        if (h % a.heads_per_group == 0) {
            for (int i = tid; i < 2 * NS; i += NT) {
                const int n = i % NS;
                const char *src = static_cast<const char *>(i < NS ? a.Bm : a.Cm) + (b * a.bcs_b + g * a.bcs_g + n) * ES;
                keep_rows(src, a.bcs_t, rows + a.nheads * kP + (i < NS ? 0 : a.ngroups * NS) + g * NS + n);
            }
        }
    }
}

struct MixPlan {
    int64_t gram, c3, b3, total;   // byte offsets of the parts, and their end
};
MixPlan mix_plan(const LaunchArgs &a) {
    const int64_t nt = (a.L + 15) / 16, np = (nt + 1) / 2, bg = static_cast<int64_t>(a.batch) * a.ngroups;
    auto up = [](int64_t v) { return (v + 255) / 256 * 256; };
    MixPlan p;
    p.gram = 0;
    p.c3 = up(bg * nt * (np + 1) * 3072);
    p.b3 = p.c3 + up(bg * nt * (a.dstate < 32 ? 1 : a.dstate / 32) * 3072);
    p.total = p.b3 + up(bg * (a.dstate / 16) * np * 3072);
    return p;
}

template <int NW, int MR, int NS, bool BF16>
hipError_t mix_head(const MixArgs &k, unsigned grid, hipStream_t s) {
    if (k.commit)
        hipLaunchKernelGGL((bdlm_mix_kernel<NW, MR, NS, BF16, true>), dim3(grid), dim3(64 * NW), 0, s, k);
    else
        hipLaunchKernelGGL((bdlm_mix_kernel<NW, MR, NS, BF16, false>), dim3(grid), dim3(64 * NW), 0, s, k);
    return hipGetLastError();
}
template <int NS, bool BF16>
hipError_t mix_launch(const MixArgs &k, hipStream_t s) {
    const int nb = (k.L + 63) / 64;
    const unsigned gg = static_cast<unsigned>(k.batch) * k.ngroups * nb * (k.y ? nb + 1 : 1);
    hipLaunchKernelGGL((bdlm_mix_gram_kernel<NS, BF16>), dim3(gg), dim3(512), 0, s, k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const unsigned grid = static_cast<unsigned>(k.batch) * k.nheads;
    if (k.L <= 64) return mix_head<4, 1, NS, BF16>(k, grid, s);
    if (k.L <= 128) return mix_head<8, 1, NS, BF16>(k, grid, s);
    return mix_head<8, 2, NS, BF16>(k, grid, s);
}
template <bool BF16>
hipError_t mix_any(const MixArgs &k, int ns, hipStream_t s) {
    switch (ns) {
        case 16: return mix_launch<16, BF16>(k, s);
        case 32: return mix_launch<32, BF16>(k, s);
        case 64: return mix_launch<64, BF16>(k, s);
        case 128: return mix_launch<128, BF16>(k, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool mix_fits(const LaunchArgs &a) {
    // the Gram tiles and the split Cf and Bf live in the caller's convolution workspace, whose
    // size is that of the convolved inputs: too small only where there are few heads per group
    // or next to no tokens
    // (rows are addressed with 31-bit byte offsets, and a launch holds fewer than 2^32 threads)
    constexpr int64_t kMax = int64_t(1) << 31;
    const int64_t es = a.bf16 ? 2 : 4, nb = (a.L + 63) / 64;
    return a.L >= 1 && a.L <= 256 && static_cast<int64_t>(a.batch) * a.ngroups * nb * (nb + 1) * 512 < 2 * kMax &&
           a.L * a.xs_t * es + 256 < kMax && a.L * a.bcs_t * es + 512 < kMax &&
           static_cast<int64_t>(a.L) * a.nheads * kP * 4 < kMax &&
           mix_plan(a).total <= conv_workspace(a.batch, a.L, a.nheads, a.ngroups, a.dstate);
}

int launch_mix(const LaunchArgs &a, const float *w, const float *bias, float *conv_pool, bool commit,
               void *ws, void *stream) {
    if (a.batch == 0 || a.L == 0) return BDLM_OK;
    if (!mix_fits(a)) return BDLM_E_SHAPE;
    if (!commit && !a.y) return BDLM_OK;
    const MixPlan p = mix_plan(a);
    char *base = static_cast<char *>(ws);
    MixArgs k;
    k.x = a.x;
    k.dt = a.dt;
    k.Bm = a.Bm;
    k.Cm = a.Cm;
    k.A = a.A;
    k.D = a.D;
    k.D_rev = a.D_rev;
    k.w = w;
    k.bias = bias;
    k.cache = conv_pool;
    k.pool = a.h_pool;
    k.y = a.y;
    k.gram = reinterpret_cast<uint4 *>(base + p.gram);
    k.c3 = reinterpret_cast<uint2 *>(base + p.c3);
    k.b3 = reinterpret_cast<uint2 *>(base + p.b3);
    k.xs_b = a.xs_b;
    k.xs_t = a.xs_t;
    k.xs_h = a.xs_h;
    k.dts_b = a.dts_b;
    k.dts_t = a.dts_t;
    k.bcs_b = a.bcs_b;
    k.bcs_t = a.bcs_t;
    k.bcs_g = a.bcs_g;
    k.L = a.L;
    k.nt = (a.L + 15) / 16;
    k.np = (k.nt + 1) / 2;
    k.batch = a.batch;
    k.nheads = a.nheads;
    k.ngroups = a.ngroups;
    k.heads_per_group = a.nheads / a.ngroups;
    k.channels = a.nheads * kP + 2 * a.ngroups * a.dstate;
    k.commit = commit ? 1 : 0;
    k.xcd_remap = (static_cast<int64_t>(a.batch) * a.nheads) % 8 == 0 ? 1 : 0;
    k.use_slots = a.slots ? 1 : 0;
    for (int i = 0; i < BDLM_MAX_SLOT_ROWS; ++i) k.slots[i] = (a.slots && i < a.batch) ? a.slots[i] : 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = a.bf16 ? mix_any<true>(k, a.dstate, s) : mix_any<false>(k, a.dstate, s);
    return e == hipSuccess ? BDLM_OK : BDLM_E_LAUNCH;
}

}  // namespace bdlm
