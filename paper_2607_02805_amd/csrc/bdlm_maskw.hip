// bdlm_maskw.hip -- gfx950 kernel for blocks of 65 to 256 tokens in the masked-matrix form of
// bdlm_mask.hip, whose header defines it, with the sources passing through LDS in windows: for
// steps whose reverse branch has its own inputs, and for one input set where windows let two
// workgroups share a CU.  bf16 activations.
//
// A step with separate reverse inputs (kSep) takes the lower triangle (j <= t, weight 1 on the
// diagonal) from the forward set, then the upper one from the reverse set; kStep and kCommit take
// both from one set, window by window.
//
// Work split: one workgroup of eight waves per (b, h); a wave owns the output rows of one
// tile (two for more than 128 tokens) of 16 tokens and all 64 head-dim columns.  A window is 128
// source tokens: row images of B and x.  For each pair of source tiles a wave forms the
// transposed Gram tiles (rows j, columns t) on bf16 MFMA from B in LDS and its own rows of C
// (registers, loaded straight from memory: dstate 32qp + 8grp .. +7 of a row is one 16-byte
// operand), weights them into the masked matrix, splits that into bf16 hi + lo and contracts it
// with x read transposed from LDS; the accumulator of the Gram product is already an operand of
// that contraction.  Products that end in y have its columns as rows, so a lane stores four
// columns of one token at once.  The prefix term contracts the same C operands with the state,
// split once per workgroup into a bf16 hi + lo image where the B window goes afterwards.
//
// A commit's state update runs over the windows before the outputs do (which then take them in
// the opposite order): its accumulators and theirs would not fit side by side.
//
// What binds it: neither unit by itself.  Four waves per SIMD, kStep at 32 x 32, 96 tokens, dstate
// 128 | kSep at 64 x 24, 128 tokens, dstate 64: the vector ALU is busy in 34 | 40 % of the cycles, the
// matrix unit in 17 | 12 %; a wave waits for memory, LDS or a barrier 40 | 49 % of its time, and for
// an issue slot, all four being at the same stage, 41 | 24 %.  Measured as graph replays, before -> here (before: kSep as a forward and
// a reverse sequence pass; one set in bdlm_mask.hip, one workgroup per CU):
//   kSep   1 row x 26 heads, 256 tokens, dstate 128   32.4 -> 25.3 us
//          8 x 32, 256 tokens, dstate 128             38.3 -> 30.0 us
//          16 x 32, 128 tokens, dstate 128            30.8 -> 22.5 us
//          64 x 24, 128 tokens, dstate 64             66.2 -> 49.8 us
//   kStep  32 x 32, 96 tokens, dstate 128             32.9 -> 25.1 us
//          16 x 24, 256 tokens, dstate 64             27.6 -> 25.8 us
// and the error against 64 bits is no larger (kSep, 256 tokens: 3.8e-8; the sequence passes 4.0e-8).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bdlm.h"
#include "bdlm_device.h"
#include "bdlm_images.h"
#include "bdlm_launch.h"

namespace bdlm {
namespace {

constexpr int kMW = 8;                 // waves per workgroup
constexpr int kMThreads = 64 * kMW;
constexpr int kWT = 128;               // tokens per source window
constexpr int kCUs = 256;              // compute units of the chip
constexpr int kStep = 0, kCommit = 1, kSep = 2;

struct WindowInputs {
    const void *x, *dt, *Bm, *Cm;      // bf16
    const float *A;
};
struct WindowArgs {
    WindowInputs in[2];                  // kSep: the forward and the reverse branch's; else in[0]
    const float *D, *D_rev;
    float *pool;                       // cached states (commit: updated in place)
    float *y;                          // outputs, or nullptr (a commit without them)
    int64_t xs_b, xs_t, xs_h;
    int64_t dts_b, dts_t;
    int64_t bcs_b, bcs_t, bcs_g;
    int32_t L, nheads, heads_per_group;
    int32_t nunits;                    // (batch row, head) units
    int32_t xcd_remap;                 // units and grid % 8 == 0: a row's units on one XCD
    int32_t use_slots;
    int32_t slots[BDLM_MAX_SLOT_ROWS];
};

constexpr uint32_t kOOB = 0x80000000u;   // offset past the resource: stores are dropped
constexpr int kNT = 2;                   // buffer cache policy: nontemporal
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), static_cast<short>(0),
                                             0x7fffffff, 0x00020000);
}
__device__ __forceinline__ float ex2(float v) { return __builtin_amdgcn_exp2f(v); }
// State quad (q, grp) of column p in the pool layout: s[p][16q + 4grp .. +3].
__device__ __forceinline__ int quad_off(int q, int grp, int p) { return ((4 * q + grp) * kP + p) * 4; }
__device__ __forceinline__ f32x4 mma_pair(uint4 a, uint4 b, f32x4 c) {
    return mma_k32(lo4(a), hi4(a), lo4(b), hi4(b), c);
}

// WIDE: registers for two waves per SIMD, so that a window's loads fly over the products of the
// one before (few workgroups: latency); else for four, two workgroups per CU.
template <int NS, int MT, int MODE, bool WIDE>
__global__ void __launch_bounds__(kMThreads) __attribute__((amdgpu_waves_per_eu(WIDE ? 2 : 4)))
bdlm_mask_window_kernel(const WindowArgs a) {
    constexpr bool COMMIT = MODE == kCommit, SEP = MODE == kSep;
    constexpr int QN = NS / 16;            // dstate tiles
    constexpr int QP = NS >= 32 ? NS / 32 : 1;   // 32-deep operands over dstate
    constexpr int TPW = MT / kMW;          // token tiles per wave
    constexpr int NTOK = 16 * MT;          // tokens of the padded block
    constexpr int TPL = NTOK / 64;         // tokens per lane in the decay scan
    constexpr int NW = NTOK / kWT;         // source windows
    constexpr int CPR = NS / 8;            // 16-byte pieces per B / C row
    constexpr int NCT = (4 * QN + kMW - 1) / kMW;   // commit tiles per wave
    constexpr int SQP = 2 * QP * 2 * 64;   // 16-byte entries of each state image (hi, lo)
    static_assert((TPW == 1 || TPW == 2) && (TPL == 2 || TPL == 4), "block tiles");
    // the state's bf16 hi and lo images, then the window's B
    __shared__ __align__(16) uint4 sU[kWT * CPR > 2 * SQP ? kWT * CPR : 2 * SQP];
    __shared__ __align__(16) uint4 sX[kWT * 8];
    __shared__ __align__(16) float sDt[NTOK], sCs[NTOK], sEx[NTOK], sEc[NTOK];
    __shared__ __align__(16) float sLa[NTOK], sLb[NTOK], sUa[NTOK], sUb[NTOK];
    __shared__ __align__(16) float sWc[COMMIT ? NTOK : 4], sDr[SEP ? NTOK : 4];
    __shared__ float2 sE[MT], sEr[SEP ? MT : 1];   // E_k in two floats
    uint4 *const sB = sU, *const sSH = sU, *const sSL = sU + SQP;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4;
    // opaque copies: LDS addresses and offsets are formed where they are used, in every
    // window, not held in registers across them
    auto opaque = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    const int L = a.L;                     // 1 <= L <= NTOK
    const bool want_y = a.y != nullptr;
    // Waves w and w + 4 share a SIMD: their rows lie as far from the block's ends, together.
    const int wrow = wave < 4 ? wave : 11 - wave;
    const int mt0 = TPW * wrow;            // first token tile of this wave's rows
    const int jpd = mt0 >> 1;              // the pair of source tiles that holds its diagonal

    // One workgroup per unit (batch row, head); with the XCD remap the units of one XCD
    // (workgroup w sits on XCD w % 8) are a contiguous run, so the heads of a row share one
    // L2.
    int v = blockIdx.x;
    if (v >= a.nunits) return;
    if (a.xcd_remap) v = (v & 7) * (a.nunits >> 3) + (v >> 3);
    const int b = v / a.nheads, h = v - b * a.nheads, g = h / a.heads_per_group;
    const int64_t slot = a.use_slots ? a.slots[b] : b;
    float *const hs = a.pool + (slot * a.nheads + h) * (kP * NS);
    auto x_of = [&](int s) { return static_cast<const uint16_t *>(a.in[s].x) + b * a.xs_b + h * a.xs_h; };
    auto dt_of = [&](int s) { return static_cast<const uint16_t *>(a.in[s].dt) + b * a.dts_b + h; };
    auto B_of = [&](int s) { return static_cast<const uint16_t *>(a.in[s].Bm) + b * a.bcs_b + g * a.bcs_g; };
    auto C_of = [&](int s) { return static_cast<const uint16_t *>(a.in[s].Cm) + b * a.bcs_b + g * a.bcs_g; };
    const uint32_t bcrow = static_cast<uint32_t>(a.bcs_t * 2), xrow = static_cast<uint32_t>(a.xs_t * 2);
    const uint32_t dtrow = static_cast<uint32_t>(a.dts_t * 2);

    // ---- loads, through buffer resources with uniform bases (rows past the block get an
    // offset past the resource's range and load zeros), in 16-byte pieces: a window's B (cached:
    // every head of the row reads it) and x, this wave's rows of C, the state in its pool layout
    constexpr int BCN = kWT * CPR, BCK = BCN >= kMThreads ? BCN / kMThreads : 1;
    constexpr int XK = kWT * 8 / kMThreads;
    constexpr int SN = 16 * NS, SK = SN >= kMThreads ? SN / kMThreads : 1;
    const bool b_own = BCN >= kMThreads || tid < BCN, s_own = SN >= kMThreads || tid < SN;
    u32x4 br[BCK], xr[XK];
    auto load_window = [&](int s, int w) {
        const __amdgpu_buffer_rsrc_t rB = rsrc(B_of(s)), rX = rsrc(x_of(s));
        const int tid = opaque(threadIdx.x);
#pragma unroll
        for (int k = 0; k < BCK; ++k) {
            const int i = tid + kMThreads * k, t = kWT * w + i / CPR;
            br[k] = __builtin_amdgcn_raw_buffer_load_b128(rB, b_own && t < L ? t * bcrow + i % CPR * 16 : kOOB, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < XK; ++k) {
            const int i = tid + kMThreads * k, t = kWT * w + (i >> 3);
            xr[k] = __builtin_amdgcn_raw_buffer_load_b128(rX, t < L ? t * xrow + (i & 7) * 16 : kOOB, 0, 0);
        }
    };
    auto stage_window = [&]() {
        const int tid = opaque(threadIdx.x);
#pragma unroll
        for (int k = 0; k < BCK; ++k) {
            const int i = tid + kMThreads * k;
            if (b_own) sB[c_at<NS>(i / CPR, i % CPR)] = __builtin_bit_cast(uint4, br[k]);
        }
#pragma unroll
        for (int k = 0; k < XK; ++k) {
            const int i = tid + kMThreads * k;
            sX[x_at(i >> 3, i & 7)] = __builtin_bit_cast(uint4, xr[k]);
        }
    };
    // this wave's rows 16 mt + col of C, an operand of its Gram tiles and of its prefix terms
    // (dstate 16: the lane groups past the row hold zeros, here and in what C meets)
    uint4 cq[TPW][QP];
    auto load_c = [&](int s) {
        const int ln = opaque(lane), col = ln & 15, grp = ln >> 4;
        const __amdgpu_buffer_rsrc_t rC = rsrc(C_of(s));
#pragma unroll
        for (int m = 0; m < TPW; ++m) {
            const int t = 16 * (mt0 + m) + col;
#pragma unroll
            for (int qp = 0; qp < QP; ++qp) {
                const bool in = t < L && (NS >= 32 || grp < 2);
                cq[m][qp] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          rC, in ? t * bcrow + (4 * qp + grp) * 16 : kOOB, 0, 0));
            }
        }
    };
    // rows j = 16 jt + col of the window's B, the other operand of the Gram tiles
    auto b_read = [&](int jt, int qp, int ln) -> uint4 {
        const int col = ln & 15, grp = ln >> 4;
        if constexpr (NS >= 32) {
            return sB[c_at<NS>(16 * jt + col, 4 * qp + grp)];
        } else {
            const uint4 r = sB[c_at<NS>(16 * jt + col, grp & 1)];
            return grp < 2 ? r : uint4{0u, 0u, 0u, 0u};
        }
    };

    // ---- the decay sums of set s (one wave, TPL tokens per lane)
    uint32_t dtraw[TPL];
    const bool scans = wave == 0 || (SEP && wave == 1);
    const int sset = SEP ? wave & 1 : 0;
    if (scans) {
        const __amdgpu_buffer_rsrc_t rD = rsrc(dt_of(sset));
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            const int t = TPL * lane + i;
            dtraw[i] = __builtin_amdgcn_raw_buffer_load_b16(rD, t < L ? t * dtrow : kOOB, 0, 0);
        }
    }
    u32x4 sr[SK];
    if (want_y) {
        const __amdgpu_buffer_rsrc_t rS = rsrc(hs);
#pragma unroll
        for (int k = 0; k < SK; ++k)
            sr[k] = __builtin_amdgcn_raw_buffer_load_b128(rS, s_own ? 16u * (tid + kMThreads * k) : kOOB, 0, COMMIT ? 0 : kNT);
        load_c(0);
    }

    if (scans) {
        // double: over 256 tokens a float's ulp of cs would show in every weight
        const double A2 = a.in[sset].A[h] * 1.4426950408889634;
        const bool fwd = !SEP || sset == 0, rev = !SEP || sset == 1;
        float dtv[TPL];
        double cs[TPL], ex[TPL], run = 0.;
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            dtv[i] = __uint_as_float(dtraw[i] << 16);
            ex[i] = run;
            run += dtv[i] * A2;
            cs[i] = run;
        }
        const double excl = wave_inclusive_sum_d(run) - run;
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            cs[i] += excl;
            ex[i] += excl;
        }
        // this lane's tile k; E_k and E_{k-1} from the lanes holding tokens 16k + 15, 16k - 1
        const int k = (TPL * lane) >> 4;
        constexpr int LPT = 16 / TPL;      // lanes per tile
        const double Ek = __shfl(cs[TPL - 1], LPT * k + LPT - 1, 64);
        const double Ekm1 = __shfl(ex[0], LPT * k, 64);
        const double Elast = __shfl(cs[TPL - 1], 63, 64);
        auto f = [](double v) { return static_cast<float>(v); };
#pragma unroll
        for (int i = 0; i < TPL; ++i) {
            const int t = TPL * lane + i;
            if (fwd) {
                sDt[t] = dtv[i];
                sCs[t] = f(cs[i] - Ekm1);   // (within the tile)
                sEc[t] = ex2(f(cs[i]));
                sLa[t] = ex2(f(cs[i] - Ekm1));
                sLb[t] = ex2(f(Ek - cs[i])) * dtv[i];
            }
            if (rev) {
                if constexpr (SEP) sDr[t] = dtv[i];
                sEx[t] = f(ex[i] - Ekm1);
                sUa[t] = ex2(f(Ek - ex[i]));
                sUb[t] = ex2(f(ex[i] - Ekm1)) * dtv[i];
            }
            if constexpr (COMMIT) sWc[t] = ex2(f(Elast - cs[i])) * dtv[i];
        }
        if ((lane & (LPT - 1)) == LPT - 1) (rev && SEP ? sEr : sE)[k] = float2{f(Ek), f(Ek - f(Ek))};
    }

    // y of this unit, transposed tiles: lane (grp, col) holds token 16 mt + col, columns 16 pt +
    // 4 grp .. +3
    f32x4 Y[TPW][4];
    if (want_y) {
        // ---- the state split into bf16 hi + lo: entry (quad pair n, column p) holds dstate 8n
        // .. 8n + 7 of column p
        uint2 *sh2 = reinterpret_cast<uint2 *>(sSH), *sl2 = reinterpret_cast<uint2 *>(sSL);
#pragma unroll
        for (int k = 0; k < SK; ++k) {
            if (!s_own) break;
            const int i = tid + kMThreads * k;             // pool-layout quad n4 * 64 + p
            s16x4 hi, lo;
            split4(__builtin_bit_cast(f32x4, sr[k]), hi, lo);
            const int at = 2 * ((i >> 7) * kP + (i & 63)) + ((i >> 6) & 1);
            sh2[at] = as_u2(hi);
            sl2[at] = as_u2(lo);
        }
        load_window(0, 0);
        __syncthreads();
        // ---- prefix term 2^{cs_t} (C_t . s^T)
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) {
#pragma unroll
            for (int m = 0; m < TPW; ++m) Y[m][pt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int qp = 0; qp < QP; ++qp) {
                const int at = (4 * qp + (NS >= 32 ? grp : grp & 1)) * kP + 16 * pt + col;
                uint4 sh = sSH[at], sl = sSL[at];
                if constexpr (NS < 32) {
                    if (grp >= 2) sh = sl = uint4{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int m = 0; m < TPW; ++m) {
                    Y[m][pt] = mma_pair(sh, cq[m][qp], Y[m][pt]);
                    Y[m][pt] = mma_pair(sl, cq[m][qp], Y[m][pt]);
                }
                if (!WIDE && (qp & 1)) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int m = 0; m < TPW; ++m) Y[m][pt] *= sEc[16 * (mt0 + m) + col];
        }
        __syncthreads();   // the images are overwritten next
    } else {
        load_window(0, 0);
    }
    stage_window();
    __syncthreads();

    if constexpr (COMMIT) {
        // ---- s_new[p, n] = 2^{cs_last} s[p, n] + sum_j B[j, n] wc_j x[j, p] on this
        // wave's tiles k = wave + 8i (columns 16 pt + col, pt = wave & 3 for every tile of the
        // wave; dstate tile k >> 2).  A operand: lane (col, grp) holds B[16 jt + 4 grp + r][16 q +
        // col], read transposed from the row image (the four quads of a dstate tile are two
        // neighbouring pieces).
        const int pt = wave & 3;
        f32x4 so[NCT];
        const float keep = ex2(sE[MT - 1].x);
#pragma unroll
        for (int i = 0; i < NCT; ++i) {
            const int k = wave + kMW * i;
            so[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (k < 4 * QN) so[i] = *reinterpret_cast<const f32x4 *>(hs + quad_off(k >> 2, grp, 16 * pt + col)) * keep;
        }
        const uint2 *sB2 = reinterpret_cast<const uint2 *>(sB);
#pragma unroll 1
        for (int w = 0; w < NW; ++w) {
            if (WIDE && w + 1 < NW) load_window(0, w + 1);
            const int lane = opaque(threadIdx.x) & 63, grp = lane >> 4;
#pragma unroll
            for (int jt = 0; jt < kWT / 16; jt += 2) {
                s16x4 wh[2], wm[2], wl[2];
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const f32x4 wc = *reinterpret_cast<const f32x4 *>(&sWc[kWT * w + 16 * (jt + d) + 4 * grp]);
                    split4x3(wc * quad_val(x_read(sX, jt + d, pt, lane)), wh[d], wm[d], wl[d]);
                }
#pragma unroll
                for (int i = 0; i < NCT; ++i) {
                    const int q = (wave + kMW * i) >> 2;
                    if (q >= QN) break;
                    s16x4 bt[2];
#pragma unroll
                    for (int d = 0; d < 2; ++d)
                        bt[d] = ds_read_tr(sB2 + 2 * c_at<NS>(16 * (jt + d) + tr_tok(lane), 2 * q + ((lane & 3) >> 1)) + (lane & 1));
                    so[i] = mma_k32(bt[0], bt[1], wh[0], wh[1], so[i]);
                    so[i] = mma_k32(bt[0], bt[1], wm[0], wm[1], so[i]);
                    so[i] = mma_k32(bt[0], bt[1], wl[0], wl[1], so[i]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (w + 1 < NW) {
                if constexpr (!WIDE) load_window(0, w + 1);
                __syncthreads();   // every wave is done with this window
                stage_window();
                __syncthreads();
            }
        }
#pragma unroll
        for (int i = 0; i < NCT; ++i) {
            const int k = wave + kMW * i;
            if (k < 4 * QN) *reinterpret_cast<f32x4 *>(hs + quad_off(k >> 2, grp, 16 * pt + col)) = so[i];
        }
    }
    if (!want_y) return;

    // This wave's rows of x for the skip term, which comes last: every product added after it
    // would round at its size.
    constexpr int NSET = SEP ? 2 : 1;
    constexpr bool EARLY = WIDE || MT == 8;   // registers for them beside the last window's
    uint2 xs[NSET][TPW][4];
    auto load_rows = [&]() {
#pragma unroll
        for (int s = 0; s < NSET; ++s) {
            const __amdgpu_buffer_rsrc_t rX = rsrc(x_of(s));
#pragma unroll
            for (int m = 0; m < TPW; ++m)
#pragma unroll
                for (int pt = 0; pt < 4; ++pt) {
                    const int t = 16 * (mt0 + m) + col;
                    xs[s][m][pt] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(
                                                                 rX, t < L ? t * xrow + 8 * grp : kOOB, 32 * pt, 0));
                }
        }
    };

    // ---- masked product: rows t of this wave's tiles, sources j window by window
    // (kSep: the forward set's windows, then the reverse set's)
    constexpr int NV = SEP ? 2 * NW : NW;
#pragma unroll 1
    for (int vis = 0; vis < NV; ++vis) {
        const int s = SEP ? vis / NW : 0;
        const int w = COMMIT ? NW - 1 - vis : (SEP ? vis % NW : vis);
        const int lane = opaque(threadIdx.x) & 63, col = lane & 15, grp = lane >> 4;
        const bool lower = !SEP || s == 0, upper = !SEP || s == 1;
        // this wave's row factors, and the tile-pair factors of its rows, lane m MT + jt:
        // 2^{E_{mt-1} - E_jt} below the diagonal, 2^{E_{jt-1} - E_mt} above it
        float la[TPW], ua[TPW], tf;
#pragma unroll
        for (int m = 0; m < TPW; ++m) {
            la[m] = sLa[16 * (mt0 + m) + col];
            ua[m] = sUa[16 * (mt0 + m) + col];
        }
        {
            const float2 *E = SEP && s == 1 ? sEr : sE;
            const int m = lane / MT, jt = lane % MT, mt = mt0 + (m < TPW ? m : 0);
            const float2 hi = E[jt < mt ? mt - 1 : (jt > mt ? jt - 1 : mt)], lo = E[jt < mt ? jt : mt];
            tf = ex2((hi.x - lo.x) + (hi.y - lo.y));
        }
        // Gram tiles of the window's source tiles 2 jp, 2 jp + 1, transposed: lane (col, grp)
        // holds G[t][j], t = 16 mt + col, j = 16 jt + 4 grp + r
        auto gram = [&](int jp, int lane, f32x4 (&gt)[2][TPW]) {
#pragma unroll
            for (int d = 0; d < 2; ++d) {
#pragma unroll
                for (int m = 0; m < TPW; ++m) gt[d][m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int qp = 0; qp < QP; ++qp) {
                    const uint4 bj = b_read(2 * jp + d, qp, lane);
#pragma unroll
                    for (int m = 0; m < TPW; ++m) gt[d][m] = mma_pair(bj, cq[m][qp], gt[d][m]);
                    if (!WIDE && (qp & 1)) __builtin_amdgcn_sched_barrier(0);   // few operands in registers at a time
                }
            }
        };
        // the weighted tiles, split (the two source tiles side by side), contracted with x
        auto contract = [&](int jp, int lane, const f32x4 (&mw)[2][TPW]) {
            uint4 mh[TPW], ml[TPW];
#pragma unroll
            for (int m = 0; m < TPW; ++m) {
                uint2 hh[2], ll[2];
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    s16x4 th, tl;
                    split4(mw[d][m], th, tl);
                    hh[d] = as_u2(th);
                    ll[d] = as_u2(tl);
                }
                mh[m] = uint4{hh[0].x, hh[0].y, hh[1].x, hh[1].y};
                ml[m] = uint4{ll[0].x, ll[0].y, ll[1].x, ll[1].y};
            }
            if constexpr (!WIDE) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
                const s16x4 x0 = x_read(sX, 2 * jp, pt, lane), x1 = x_read(sX, 2 * jp + 1, pt, lane);
#pragma unroll
                for (int m = 0; m < TPW; ++m) {
                    Y[m][pt] = mma_k32(x0, x1, lo4(mh[m]), hi4(mh[m]), Y[m][pt]);
                    Y[m][pt] = mma_k32(x0, x1, lo4(ml[m]), hi4(ml[m]), Y[m][pt]);
                }
            }
        };
        constexpr int WP = kWT / 32;       // source pairs per window
        const int vn = vis + 1, sn = SEP ? vn / NW : 0, wn = COMMIT ? NW - 1 - vn : (SEP ? vn % NW : vn);
        if (WIDE && vn < NV) load_window(sn, wn);
        if constexpr (EARLY) {
            if (vn == NV) load_rows();
        }
        const int p0 = SEP && !lower ? (jpd + 1 - WP * w > 0 ? jpd + 1 - WP * w : 0) : 0;
        const int p1 = SEP && lower ? (jpd - WP * w < WP ? jpd - WP * w : WP) : WP;
#pragma unroll 1
        for (int jp = p0; jp < p1; ++jp) {
            const int j0 = kWT / 16 * w + 2 * jp;   // the first source tile, in the block
            if (j0 == 2 * jpd) continue;            // the diagonal's pair follows
            const bool below = j0 < mt0;
            f32x4 gt[2][TPW];
            gram(jp, lane, gt);
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const f32x4 fac = *reinterpret_cast<const f32x4 *>((below ? sLb : sUb) + 16 * (j0 + d) + 4 * grp);
#pragma unroll
                for (int m = 0; m < TPW; ++m) {
                    const float sf = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tf), m * MT + j0 + d));
                    gt[d][m] *= fac * ((below ? la[m] : ua[m]) * sf);
                }
            }
            contract(jp, lane, gt);
        }
        if (jpd >= WP * w && jpd < WP * (w + 1)) {
            // the pair of source tiles with the diagonal tiles (both branches, and the token's own
            // input twice, or one of them); the tiles beside them are one boundary away
            const int jp = jpd - WP * w, lane = opaque(threadIdx.x) & 63, col = lane & 15, grp = lane >> 4;
            const float *dts = SEP && s == 1 ? sDr : sDt;
            f32x4 gt[2][TPW];
            gram(jp, lane, gt);
#pragma unroll
            for (int m = 0; m < TPW; ++m) {
                const int mt = mt0 + m, t = 16 * mt + col;
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const int jt = 2 * jpd + d, j = 16 * jt + 4 * grp;
                    f32x4 w4;
                    if (jt < mt) {
                        w4 = *reinterpret_cast<const f32x4 *>(&sLb[j]) * la[m];
                    } else if (jt > mt) {
                        w4 = *reinterpret_cast<const f32x4 *>(&sUb[j]) * ua[m];
                    } else {
                        const float cst = sCs[t], ext = sEx[t];
                        const f32x4 csj = *reinterpret_cast<const f32x4 *>(&sCs[j]);
                        const f32x4 exj = *reinterpret_cast<const f32x4 *>(&sEx[j]);
                        const f32x4 dtj = *reinterpret_cast<const f32x4 *>(&dts[j]);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int i = 4 * grp + r;   // positions within the tile
                            const float e = ex2(i < col ? cst - csj[r] : exj[r] - ext);
                            w4[r] = (i == col ? (SEP ? 1.f : 2.f) : e) * dtj[r];
                        }
                    }
                    gt[d][m] *= w4;
                    if constexpr (SEP) {   // the other triangle has no part, whatever its operands hold
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (j + r < t ? !lower : (j + r > t && !upper)) gt[d][m][r] = 0.f;
                    }
                }
            }
            contract(jp, lane, gt);
        }
        if (vn < NV) {
            if constexpr (!WIDE) load_window(sn, wn);
            if (SEP && vn == NW) load_c(1);
            __syncthreads();   // every wave is done with this window
            stage_window();
            __syncthreads();
        }
    }

    // ---- skip term and store (tokens past the block are dropped): through the cache, so a row's
    // four 64-byte pieces (pt) meet in L2
    if constexpr (!EARLY) load_rows();
    const float skip[2] = {SEP ? a.D[h] : a.D[h] + a.D_rev[h], SEP ? a.D_rev[h] : 0.f};
    const __amdgpu_buffer_rsrc_t rY = rsrc(a.y + ((static_cast<int64_t>(b) * L) * a.nheads + h) * kP);   // uniform base
    const uint32_t ytokB = static_cast<uint32_t>(a.nheads) * kP * 4;
#pragma unroll
    for (int m = 0; m < TPW; ++m) {
        const int t = 16 * (mt0 + m) + col;
        const uint32_t yo = t < L ? t * ytokB + 16 * grp : kOOB;
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) {
#pragma unroll
            for (int s = 0; s < NSET; ++s) Y[m][pt] += skip[s] * quad_val(as_s16x4(xs[s][m][pt]));
            // (the whole offset per lane: a 16-byte store whose offset is partly in a scalar register
            // may still be reading its data while the next instruction overwrites them, and the
            // compiler leaves no wait state there)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, Y[m][pt]), rY, yo + 64 * pt, 0, 0);
        }
    }
}

template <int NS, int MT, int MODE, bool WIDE>
hipError_t launch(const WindowArgs &k, hipStream_t s) {
    hipLaunchKernelGGL((bdlm_mask_window_kernel<NS, MT, MODE, WIDE>), dim3(k.nunits), dim3(kMThreads), 0, s, k);
    return hipGetLastError();
}
template <int NS>
hipError_t launch_sep(const WindowArgs &k, hipStream_t s) {
    const bool wide = k.nunits <= kCUs;
    if (k.L <= 128) return wide ? launch<NS, 8, kSep, true>(k, s) : launch<NS, 8, kSep, false>(k, s);
    if constexpr (NS < 128) {
        if (!wide) return launch<NS, 16, kSep, false>(k, s);
    }
    return launch<NS, 16, kSep, true>(k, s);
}

WindowArgs window_args(const LaunchArgs &a, const LaunchArgs &r, bool want_y) {
    WindowArgs k;
    k.in[0] = WindowInputs{a.x, a.dt, a.Bm, a.Cm, a.A};
    k.in[1] = WindowInputs{r.x, r.dt, r.Bm, r.Cm, r.A};
    k.D = a.D;
    k.D_rev = r.D_rev;
    k.pool = a.h_pool;
    k.y = want_y ? a.y : nullptr;
    k.xs_b = a.xs_b;
    k.xs_t = a.xs_t;
    k.xs_h = a.xs_h;
    k.dts_b = a.dts_b;
    k.dts_t = a.dts_t;
    k.bcs_b = a.bcs_b;
    k.bcs_t = a.bcs_t;
    k.bcs_g = a.bcs_g;
    k.L = a.L;
    k.nheads = a.nheads;
    k.heads_per_group = a.nheads / a.ngroups;
    k.use_slots = a.slots ? 1 : 0;
    for (int i = 0; i < BDLM_MAX_SLOT_ROWS; ++i) k.slots[i] = (a.slots && i < a.batch) ? a.slots[i] : 0;
    k.nunits = static_cast<int32_t>(static_cast<int64_t>(a.batch) * a.nheads);
    k.xcd_remap = k.nunits % 8 == 0 ? 1 : 0;
    return k;
}

}  // namespace

// One input set: where the whole block's images leave room for one workgroup per CU (dstate
// 128 to 128 tokens: 86 KB; dstate 64 beyond: 90 KB) and there are more workgroups than CUs.
// With fewer the whole images are faster (8 rows x 32 heads, 128 tokens: 10.0 us, windows 11.4),
// as at dstate 128 beyond 128 tokens at any number (16 x 26, 256 tokens, step and commit: 71.6
// and 75.9).
bool masked_windows_fit(const LaunchArgs &a) {
    return long_masked_fits(a) && static_cast<int64_t>(a.batch) * a.nheads > kCUs &&
           a.dstate == (a.L <= 128 ? 128 : 64);
}

int launch_masked_windows(const LaunchArgs &a, bool commit, bool want_y, void *stream) {
    const WindowArgs k = window_args(a, a, want_y);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = a.L <= 128 ? (commit ? launch<128, 8, kCommit, false>(k, s) : launch<128, 8, kStep, false>(k, s))
                                    : (commit ? launch<64, 16, kCommit, false>(k, s) : launch<64, 16, kStep, false>(k, s));
    return e == hipSuccess ? BDLM_OK : BDLM_E_LAUNCH;
}

// Separate reverse inputs: every block of 65 to 128 tokens that fits (windows over the two
// sequence passes 0.65 to 0.91).  Beyond, the block is padded to 256 tokens, where the passes walk
// 64-token chunks and at dstate 64 and less three or more of their workgroups share a CU; windows
// over passes, of 193 to 256 tokens | of 129 to 192 (32 heads):
//   dstate 128  to 256 row-heads 0.8; beyond, four waves per SIMD leave too few registers to load
//               ahead (16 x 26 x 256 tokens: 47.7 us, the passes 46.6)
//   dstate 64   to 768 row-heads 0.82 to 0.99, to 1,536 0.97 to 1.07, from 2,048 0.90 to 1.04
//               | to 256 0.97 to 1.03, beyond 1.0 to 1.29
//   dstate 32   to 512 0.82 to 0.93, to 1,536 0.96 to 1.08, from 2,048 0.88 to 1.08
//               | to 256 0.97 to 1.03, to 512 1.0 to 1.05, beyond 1.10 to 1.29
//   dstate 16   to 512 0.89 to 1.03, beyond 1.03 to 1.20 | 1.07 to 1.47
bool sep_windows_fit(const LaunchArgs &a) {
    if (!long_masked_fits(a)) return false;
    if (a.L <= 128) return true;
    const int64_t units = static_cast<int64_t>(a.batch) * a.nheads;
    if (a.dstate == 128) return units <= kCUs;
    if (a.L <= 192) return a.dstate >= 32 && units <= kCUs;
    return units <= (a.dstate == 64 ? 768 : 512) || (a.dstate >= 32 && units >= 2048);
}

int launch_block_long_sep(const LaunchArgs &fwd, const LaunchArgs &rev, void *stream) {
    if (fwd.batch == 0 || fwd.L == 0) return BDLM_OK;
    if (!sep_windows_fit(fwd)) return launch_block_long(fwd, rev, false, true, stream);
    const WindowArgs k = window_args(fwd, rev, true);
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    switch (fwd.dstate) {
        case 16: e = launch_sep<16>(k, s); break;
        case 32: e = launch_sep<32>(k, s); break;
        case 64: e = launch_sep<64>(k, s); break;
        default: e = launch_sep<128>(k, s); break;
    }
    return e == hipSuccess ? BDLM_OK : BDLM_E_LAUNCH;
}

}  // namespace bdlm
