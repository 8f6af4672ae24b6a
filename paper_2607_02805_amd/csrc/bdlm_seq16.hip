// bdlm_seq16.hip -- the sequence kernels for bf16 activations: seg_state and seg_out of
// bdlm_seq.hip, whose header says what they compute and how a sequence is cut into segments
// and 64-token chunks (fp32 activations run on the kernels there).
//
// Per chunk, with l_i = dt_i A_h log2(e), inclusive sums cs_i, ex_i = cs_i - l_i and tot = cs_63:
//   kFwd   y_i = 2^{cs_i} (C_i . S) + sum_{j<=i} 2^{cs_i - cs_j} dt_j (C_i . B_j) x_j + skip x_i
//   kBoth  kFwd plus the reverse branch's terms whose source lies in the same chunk,
//          sum_{j>=i} 2^{ex_j - ex_i} dt_j (C_i . B_j) x_j: both triangles of one masked product
//          (weight 2 on the diagonal), as in a block step
//   kPre   what is then left of the reverse branch, 2^{cs_i} (C_i . S) on the time-reversed
//          sequence (chunks walked backwards and loaded flipped), added onto y
//   S  <- 2^{tot} S + sum_j 2^{tot - cs_j} dt_j x_j (outer) B_j
// A full window runs kBoth then kPre: the C.B^T tiles, their decay weights and their splits are
// formed once per chunk instead of once per direction.
//
// Work split: four waves per head, wave w owning head-dim columns 16w .. 16w+15 of the state and
// of y; one or two heads per workgroup (HPW), which share a chunk's images of B and C and the
// C.B^T products.  A chunk is staged once in LDS as row images; operands over dstate of C are
// 16-byte reads, operands over tokens LDS transpose reads.  Rows of the state's tile q hold
// dstate 32 (q/2) + 8 grp + 4 (q%2) + r, so that a pair of tiles is one 16-byte piece of a row of
// C.  Products that end in y have its columns as rows, so a lane holds four columns of one token.
//
// Measured (4 rows of 65,536 tokens, 32 heads, dstate 128, traced): kBoth 1.25 ms with two heads
// per workgroup at four waves per SIMD, 1.38 ms with one; kPre 1.36 ms (5.5 GB, 4.0 TB/s: its
// read and second write of y bind it); a forward and a reverse pass before: 1.41 + 1.54 ms.
// kBoth is bound by issue: its vector ALU and matrix instructions take 94 % of a SIMD's cycles
// one after the other.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bdlm.h"
#include "bdlm_device.h"
#include "bdlm_images.h"
#include "bdlm_launch.h"
#include "bdlm_seq.h"

namespace bdlm {
namespace {

constexpr int kC = 64;           // chunk length (tokens): one token per lane in the scan
constexpr int kThreads = 256;    // 4 waves
constexpr int kFwd = 0, kBoth = 1, kPre = 2;

__device__ __forceinline__ float ex2(float v) { return __builtin_amdgcn_exp2f(v); }

// Decode the workgroup into (batch row, segment, head): consecutive units of one
// (row, segment) share B and C, so they are kept on one XCD.
struct Unit {
    int b, seg, h;   // h: the workgroup's first head
};
template <int HPW>
__device__ __forceinline__ Unit decode(const SeqArgs &a) {
    int u = blockIdx.x;
    if (a.xcd_remap) u = (u & 7) * (static_cast<int>(gridDim.x) >> 3) + (u >> 3);
    Unit r;
    const int nh = a.nheads / HPW;
    r.h = u % nh * HPW;
    const int rest = u / nh;
    r.seg = rest % a.nseg;
    r.b = rest / a.nseg;
    return r;
}
// Slot of workgroup (row, head, segment)'s states in ws (times dirs states each).
__device__ __forceinline__ int64_t state_slot(const SeqArgs &a, int b, int h, int seg) {
    return a.blk_major ? (static_cast<int64_t>(b) * a.nseg + seg) * a.nheads + h
                       : (static_cast<int64_t>(b) * a.nheads + h) * a.nseg + seg;
}

// Buffer resources over the first `bytes` bytes: a load past them returns zeros and a store
// there is dropped (the range check covers the per-lane offset, not the scalar one).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_n(const void *base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), static_cast<short>(0), bytes, 0x00020000);
}
constexpr uint32_t kOOB = 0x80000000u;   // offset past every resource
constexpr int kNT = 2;   // buffer cache policy: nontemporal

// B image: 8-byte quad (state tile q, lane group a) of token t.  The four quads of a tile lie side by
// side (a transpose read takes them from four tokens at once), whatever dstate they hold.
template <int NS>
__device__ __forceinline__ int b_at(int t, int q, int a) {
    constexpr int QN = NS / 16;
    return t * (NS / 4) + ((q ^ ((t / (8 / QN)) & (QN - 1))) * 4) + (a ^ (2 * ((t >> 3) & 1)));
}
// Dstate quad (of four) that tile q's rows 4 grp .. 4 grp + 3 hold, and the offset of those
// values of column p in the pool layout.
template <int NS>
__device__ __forceinline__ int n4_of(int q, int grp) { return NS >= 32 ? 8 * (q >> 1) + 2 * grp + (q & 1) : grp; }
template <int NS>
__device__ __forceinline__ int quad_off(int q, int grp, int p) { return (n4_of<NS>(q, grp) * kP + p) * 4; }

// One chunk's global loads into registers and their staging into LDS.  Local token i is row
// i of the chunk, or (REV) row 63 - i; rows past the segment have dt = 0 (decay 1, no input),
// which changes nothing, and load as zeros (at token strides shorter than a row, 0 among them, as
// parts of valid rows).
template <int NS, int HPW, bool REV, bool LOADC>
struct Stager {
    static constexpr int NT = kThreads * HPW;                          // threads
    static constexpr int CH = NS / 8;                                  // pieces per B / C row
    static constexpr int K = kC * CH >= NT ? kC * CH / NT : 1;
    static constexpr int RS = NT / CH;                                 // rows per pass
    const char *xg, *dtg, *Bg, *Cg;  // this (row, head / group) at token 0
    int64_t xrow, dtrow, bcrow;      // bytes between consecutive tokens
    int64_t s0, s1;
    int cstride;                     // tokens per chunk (64; forward: any <= 64)
    u32x4 rb[K], rc[LOADC ? K : 1], rx[2];
    uint32_t dtraw;

    __device__ __forceinline__ static int row(int i) { return REV ? kC - 1 - i : i; }
    __device__ __forceinline__ int64_t window(int c) const { return s0 + static_cast<int64_t>(cstride) * c; }
    __device__ __forceinline__ int valid(int c) const {
        const int64_t v = s1 - window(c);
        return v < cstride ? static_cast<int>(v) : cstride;
    }
    __device__ __forceinline__ int nchunks() const { return static_cast<int>((s1 - s0 + cstride - 1) / cstride); }

    // hd: the head of the workgroup that this thread's wave works on (its x and dt)
    __device__ __forceinline__ void setup(const SeqArgs &a, const Unit &un, int hd, int g) {
        xg = static_cast<const char *>(a.x) + (un.b * a.xs_b + (un.h + hd) * a.xs_h) * 2;
        dtg = static_cast<const char *>(a.dt) + (un.b * a.dts_b + un.h + hd) * 2;
        Bg = static_cast<const char *>(a.Bm) + (un.b * a.bcs_b + g * a.bcs_g) * 2;
        Cg = a.Cm ? static_cast<const char *>(a.Cm) + (un.b * a.bcs_b + g * a.bcs_g) * 2 : nullptr;
        xrow = a.xs_t * 2;
        dtrow = a.dts_t * 2;
        bcrow = a.bcs_t * 2;
        s0 = static_cast<int64_t>(un.seg) * a.S;
        s1 = s0 + a.S < a.T ? s0 + a.S : a.T;
        cstride = REV ? kC : a.cstride;
    }
    // (scan: this wave scans its head's decays)
    __device__ __forceinline__ void issue(int c, int tid, bool scan) {
        const int64_t w = window(c);
        const int lim = valid(c);
        const int bcn = static_cast<int>((lim - 1) * bcrow) + 2 * NS, xn = static_cast<int>((lim - 1) * xrow) + 2 * kP;
        const __amdgpu_buffer_rsrc_t rB = rsrc_n(Bg + w * bcrow, bcn);
        const __amdgpu_buffer_rsrc_t rC = rsrc_n(Cg + w * bcrow, bcn);
        const __amdgpu_buffer_rsrc_t rX = rsrc_n(xg + w * xrow, xn);
        const int bs = static_cast<int>((REV ? -RS : RS) * bcrow), xs = static_cast<int>((REV ? -32 : 32) * xrow);
        // (rows are at most 16 MiB: a chunk's byte offsets fit in 31 bits)
        const uint32_t ob = row(tid / CH) * static_cast<uint32_t>(bcrow) + (tid % CH) * 16;
        const uint32_t ox = row((tid & (kThreads - 1)) >> 3) * static_cast<uint32_t>(xrow) + (tid & 7) * 16;
        if (kC * CH >= NT || tid < kC * CH) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                rb[k] = __builtin_amdgcn_raw_buffer_load_b128(rB, ob + k * bs, 0, 0);
                if constexpr (LOADC) rc[k] = __builtin_amdgcn_raw_buffer_load_b128(rC, ob + k * bs, 0, 0);
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) rx[k] = __builtin_amdgcn_raw_buffer_load_b128(rX, ox + k * xs, 0, 0);
        if (scan) {
            // (a lane mask: a comparison would hold the lane number in a register)
            const bool in = __builtin_amdgcn_inverse_ballot_w64(REV ? ~0ull << (kC - lim) : ~0ull >> (kC - lim));
            const uint32_t o = in ? row(tid & 63) * static_cast<uint32_t>(dtrow) : kOOB;
            dtraw = __builtin_amdgcn_raw_buffer_load_b16(rsrc_n(dtg + w * dtrow, 0x7fffffff), o, 0, 0);
        }
    }
    __device__ __forceinline__ float dt_value() const { return __uint_as_float(dtraw << 16); }
    __device__ __forceinline__ void stage(int tid, uint2 *sB, uint4 *sC, uint4 *sX) const {
        if (kC * CH >= NT || tid < kC * CH) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                // piece c: the quads of lane group c % 4 in tiles 2 (c / 4) and 2 (c / 4) + 1, or (one
                // tile) of lane groups 2c and 2c + 1
                const int t = tid / CH + RS * k, c = tid % CH;
                sB[NS >= 32 ? b_at<NS>(t, 2 * (c >> 2), c & 3) : b_at<NS>(t, 0, 2 * c)] = uint2{rb[k].x, rb[k].y};
                sB[NS >= 32 ? b_at<NS>(t, 2 * (c >> 2) + 1, c & 3) : b_at<NS>(t, 0, 2 * c + 1)] = uint2{rb[k].z, rb[k].w};
                if constexpr (LOADC) sC[c_at<NS>(t, c)] = __builtin_bit_cast(uint4, rc[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) sX[x_at(((tid & (kThreads - 1)) >> 3) + 32 * k, tid & 7)] = __builtin_bit_cast(uint4, rx[k]);
    }
};

// B operand over tokens: lane (grp, col) gets tokens 16 jt + 4 grp .. +3 of the dstate index that
// row col of tile q holds.
template <int NS>
__device__ __forceinline__ s16x4 bt_read(const uint2 *sB, int jt, int q, int lane) {
    return ds_read_tr(sB + b_at<NS>(16 * jt + tr_tok(lane), q, lane & 3));
}

// Weighted x operands of a state update: bf16 hi + lo, or hi + mid + lo (T3) where the updated
// state leaves the kernels (a cache, the states entering blocks): carried over many blocks, a
// two-term split's 2^-18 residual per input adds up to more than the parity bar allows on
// states near zero.
template <bool T3> struct WOps { s16x4 h[4], l[4], m[T3 ? 4 : 1]; };
template <bool T3>
__device__ __forceinline__ void w_set(WOps<T3> &o, int jt, f32x4 v) {
    if constexpr (T3) split4x3(v, o.h[jt], o.m[jt], o.l[jt]);
    else split4(v, o.h[jt], o.l[jt]);
}
// acc += B^T (weighted x) over token tiles jt, jt + 1
template <bool T3>
__device__ __forceinline__ f32x4 w_mma(s16x4 b0, s16x4 b1, const WOps<T3> &w, int jt, f32x4 acc) {
    acc = mma_k32(b0, b1, w.h[jt], w.h[jt + 1], acc);
    acc = mma_k32(b0, b1, w.l[jt], w.l[jt + 1], acc);
    if constexpr (T3) acc = mma_k32(b0, b1, w.m[jt], w.m[jt + 1], acc);
    return acc;
}
// ------------------------------------------------------------------ seg_state
// Local forward state F (and, BOTH, reverse state R) of one segment from zero, and
// the segment's total log2-decay.
template <int NS, bool BOTH>
__global__ void __launch_bounds__(kThreads, 3) bdlm_seg_state16_kernel(const SeqArgs a) {
    constexpr int QN = NS / 16;
    constexpr bool T3 = !BOTH;   // forward-only segment states become cached or emitted states
    __shared__ __align__(16) uint2 sB[kC * NS / 4];
    __shared__ __align__(16) uint4 sX[kC * 8];
    __shared__ __align__(16) float sWs[kC], sWr[kC], sTot[4];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, grp = lane >> 4, p = 16 * wave + col;
    const Unit un = decode<1>(a);
    Stager<NS, 1, false, false> st;
    st.setup(a, un, 0, un.h / a.heads_per_group);
    const int nch = st.nchunks();
    const float A2 = a.A[un.h] * kLog2e;

    f32x4 F[QN], R[BOTH ? QN : 1];
#pragma unroll
    for (int q = 0; q < QN; ++q) {
        F[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (BOTH) R[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float off = 0.f;   // log2-decay of the segment's tokens before the current chunk
    st.issue(0, tid, wave == 0);
    for (int c = 0; c < nch; ++c) {
        st.stage(tid, sB, nullptr, sX);
        if (wave == 0) {
            const float dtv = st.dt_value(), l2 = dtv * A2, cs = wave_inclusive_sum(l2);
            const float tot = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cs), 63));
            sWs[lane] = ex2(tot - cs) * dtv;
            if constexpr (BOTH) sWr[lane] = ex2(cs - l2) * dtv;   // relative to the chunk's start
            if (lane == 0) sTot[0] = tot;
        }
        __syncthreads();
        if (c + 1 < nch) st.issue(c + 1, tid, wave == 0);
        const float tot = sTot[0];
        WOps<T3> wf, wr;
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
            const f32x4 xv = quad_val(x_read(sX, jt, wave, lane));
            w_set(wf, jt, *reinterpret_cast<const f32x4 *>(&sWs[16 * jt + 4 * grp]) * xv);
            if constexpr (BOTH)
                w_set(wr, jt, *reinterpret_cast<const f32x4 *>(&sWr[16 * jt + 4 * grp]) * xv * ex2(off));
        }
        const float keep = ex2(tot);
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            s16x4 b[4];
#pragma unroll
            for (int jt = 0; jt < 4; ++jt) b[jt] = bt_read<NS>(sB, jt, q, lane);
            F[q] = w_mma(b[2], b[3], wf, 2, w_mma(b[0], b[1], wf, 0, F[q] * keep));
            if constexpr (BOTH) R[q] = w_mma(b[2], b[3], wr, 2, w_mma(b[0], b[1], wr, 0, R[q]));
            __builtin_amdgcn_sched_barrier(0);
        }
        off += tot;
        __syncthreads();   // LDS is rewritten by the next chunk
    }

    float *out = a.ws + state_slot(a, un.b, un.h, un.seg) * a.dirs * (kP * NS);
#pragma unroll
    for (int q = 0; q < QN; ++q) {
        *reinterpret_cast<f32x4 *>(out + quad_off<NS>(q, grp, p)) = F[q];
        if constexpr (BOTH) *reinterpret_cast<f32x4 *>(out + kP * NS + quad_off<NS>(q, grp, p)) = R[q];
    }
    if (tid == 0) a.tot[(static_cast<int64_t>(un.b) * a.nheads + un.h) * a.nseg + un.seg] = off;
}

// ------------------------------------------------------------------ seg_out
// MODE: what is computed (header).  T3: the carried state is written out (a cache commit), so
// its updates use three-term splits.
template <int NS, int HPW, int MODE, bool T3>
__global__ void __launch_bounds__(kThreads * HPW, HPW == 2 ? 4 : (MODE == kPre ? 3 : 2)) bdlm_seg_out16_kernel(const SeqArgs a) {
    constexpr bool REV = MODE == kPre, GRAM = MODE != kPre, FULL = MODE == kBoth;
    static_assert(!(REV && T3), "the reverse pass keeps no state");
    constexpr int QN = NS / 16, CH = NS / 8;
    constexpr int NTILE = FULL ? 16 : 10;                        // tiles of M
    constexpr int TPW = FULL ? 4 / HPW : (HPW == 2 ? 2 : 3);     // products of them per wave, at most
    __shared__ __align__(16) uint2 sB[kC * 2 * CH];
    __shared__ __align__(16) uint4 sC[kC * CH], sXh[HPW][kC * 8];
    // two heads, FULL, dstate 128: M of head 0 takes C's place once every wave has read C
    constexpr bool OVER = HPW == 2 && FULL && NS == 128;
    __shared__ __align__(16) uint4 sMh[OVER ? 1 : HPW][GRAM ? (FULL ? 8 : 6) * 128 : 1];
    struct Decays {
        float Dt[kC], Cs[kC], Ec[kC], Ws[kC], La[kC], Lb[kC], Ex[FULL ? kC : 4], Ua[FULL ? kC : 4], Ub[FULL ? kC : 4];
    };
    __shared__ __align__(16) Decays sD[HPW];

    const int tid0 = threadIdx.x, lane0 = tid0 & 63;
    const int wave8 = __builtin_amdgcn_readfirstlane(tid0 >> 6);
    const int hd = HPW == 2 ? wave8 >> 2 : 0, wave = wave8 & 3;   // this wave's head, its columns
    Unit un = decode<HPW>(a);
    Stager<NS, HPW, REV, true> st;
    st.setup(a, un, hd, un.h / a.heads_per_group);
    un.h += hd;
    const int nch = st.nchunks();
    // M in LDS: source tiles in pairs, the hi quads of both as one operand, then the lo quads; the
    // first quad of tile (mt, jt), in 8-byte units
    auto m_at = [](int mt, int jt) {
        return ((FULL ? 2 * mt : (mt >> 1) * ((mt >> 1) + 1) + (mt & 1) * ((mt >> 1) + 1)) + (jt >> 1)) * 256 + (jt & 1);
    };
    auto m_of = [&](int h) -> uint4 * { return OVER ? (h == 0 ? sC : sMh[0]) : sMh[h]; };
    uint4 *const sX = sXh[hd], *const sM = m_of(hd);
    float *const sCs = sD[hd].Cs, *const sDt = sD[hd].Dt, *const sEc = sD[hd].Ec, *const sWs = sD[hd].Ws;
    const float A2 = a.A[un.h] * kLog2e;
    const float skip = MODE == kPre ? 0.f : a.skip[un.h] + (FULL ? a.skip2[un.h] : 0.f);

    // the state entering the segment (in this direction's scan order)
    auto s_off = [&](int q) { return quad_off<NS>(q, lane0 >> 4, 16 * wave + (lane0 & 15)); };
    f32x4 S[QN];
    const int64_t cslot = a.use_slots ? a.slots[un.b] : un.b;
    const float *src = a.pool_in ? a.pool_in + (cslot * a.nheads + un.h) * (kP * NS)
                                 : a.ws + (state_slot(a, un.b, un.h, un.seg) * a.dirs + (REV ? 1 : 0)) * (kP * NS);
    if (a.pool_in || !a.zero_init) {
#pragma unroll
        for (int q = 0; q < QN; ++q) S[q] = *reinterpret_cast<const f32x4 *>(src + s_off(q));
    } else {
#pragma unroll
        for (int q = 0; q < QN; ++q) S[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // The state loads complete here, before the chunk loop: otherwise the first use of each
    // quad in every chunk waits on the vector-memory counter, i.e. for the next chunk's
    // prefetched inputs.
#pragma unroll
    for (int q = 0; q < QN; ++q) asm volatile("" : "+v"(S[q]));

    // y of this (row, head) at token 0 and bytes between tokens; this lane's 16 bytes of a chunk's
    // row tile mt (local token 16 mt + col, columns 16 wave + 4 grp .. +3)
    const float *ybase = a.y + (static_cast<int64_t>(un.b) * a.T * a.nheads + un.h) * kP;
    const int64_t ytokB = static_cast<int64_t>(a.nheads) * kP * 4;

    st.issue(REV ? nch - 1 : 0, tid0, wave == 0);
    for (int k = 0; k < nch; ++k) {
        const int c = REV ? nch - 1 - k : k;
        // opaque: addresses and offsets are formed in every chunk, not held in registers across them
        int tid = tid0;
        if constexpr (HPW == 2 || MODE == kPre) asm volatile("" : "+v"(tid));
        const int lane = tid & 63, col = lane & 15, grp = lane >> 4;
        st.stage(tid, sB, sC, sX);
        if (wave == 0) {
            float *const sLa = sD[hd].La, *const sLb = sD[hd].Lb, *const sEx = sD[hd].Ex, *const sUa = sD[hd].Ua,
                        *const sUb = sD[hd].Ub;
            // the chunk's decay sums and weights; E_k is cs at the end of token tile k
            const float dtv = st.dt_value(), l2 = dtv * A2, cs = wave_inclusive_sum(l2);
            auto at = [&](int i) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cs), i)); };
            const float E0 = at(15), E1 = at(31), E2 = at(47), E3 = at(63);
            sEc[lane] = ex2(cs);
            sWs[lane] = ex2(E3 - cs) * dtv;
            sCs[lane] = cs;
            if constexpr (GRAM) {
                const float E = grp == 0 ? E0 : (grp == 1 ? E1 : (grp == 2 ? E2 : E3));
                const float Em = grp == 0 ? 0.f : (grp == 1 ? E0 : (grp == 2 ? E1 : E2));
                sDt[lane] = dtv;
                // j < t in earlier tiles: 2^{cs_t - cs_j} = sLa[t] 2^{E_{mt-1} - E_jt} sLb[j] / dt_j; j > t
                // in later ones: 2^{ex_j - ex_t} = sUa[t] 2^{E_{jt-1} - E_mt} sUb[j] / dt_j
                sLa[lane] = ex2(cs - Em);
                sLb[lane] = ex2(E - cs) * dtv;
                if constexpr (FULL) {
                    // the exclusive sum is the token before's inclusive one (not cs - l2, which would
                    // round once more at the sum's size: a third of the weights' error)
                    const float ex = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(cs), 0x138, 0xf, 0xf, true));
                    sEx[lane] = ex;
                    sUa[lane] = ex2(E - ex);
                    sUb[lane] = ex2(ex - Em) * dtv;
                }
            }
        }
        __syncthreads();
        if constexpr (!GRAM && HPW == 1) {
            if (k + 1 < nch) st.issue(REV ? c - 1 : c + 1, tid, wave == 0);
        }
        // (rows past the segment lie past the resource's range)
        const __amdgpu_buffer_rsrc_t rY =
            rsrc_n(ybase + st.window(c) * (ytokB / 4), static_cast<int>(st.valid(c) * ytokB));
        const uint32_t oy = Stager<NS, HPW, REV, true>::row(col) * static_cast<uint32_t>(ytokB) + (16 * wave + 4 * grp) * 4;
        auto y_off = [&](int mt) { return oy + static_cast<uint32_t>((REV ? -16 : 16) * mt * ytokB); };
        // the passes that add onto y request this lane's values now (one reader and writer per
        // element: the sum is exact fp32 and deterministic)
        f32x4 yv[REV ? 4 : 1];
        if constexpr (REV) {
            if (a.y) {
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
                    yv[mt] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rY, y_off(mt), 0, 0));
            }
        }

        // ---- decay-weighted C.B^T tiles M[t][j], held as the transposed product (lane (grp, col):
        // j = 16jt + 4grp + r, t = 16mt + col) and split: FULL wave w takes row tile w, else tiles
        // w, w + 4, w + 8 of the lower triangle
        f32x4 g[GRAM ? TPW : 1];
        int mt[GRAM ? TPW : 1], jt[GRAM ? TPW : 1], kt[GRAM ? TPW : 1], h0[GRAM ? TPW : 1], h1[GRAM ? TPW : 1];
        if constexpr (GRAM) if (a.y) {
            int wv = wave8;   // opaque: the tiles' LDS addresses are formed here, not held in
            asm volatile("" : "+s"(wv));   // registers across the loop
            // Product i is tile kt = row tile mt, source tile jt, weighted for heads [h0, h1).  One
            // head: FULL row tile w in wave w, else tiles w, w + 4, w + 8 of the lower triangle.  Two
            // heads share each product: FULL half of row tile w % 4 in wave w; else tile w, and tiles 8
            // and 9 in waves 0 to 3, one head each.
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                h0[i] = 0;
                h1[i] = HPW;
                if constexpr (FULL) {
                    mt[i] = wv & 3;
                    jt[i] = TPW * (wv >> 2) + i;
                    kt[i] = 4 * mt[i] + jt[i];
                } else {
                    kt[i] = HPW == 1 ? wv + 4 * i : (i == 0 ? wv : 8 + ((wv >> 1) & 1));
                    if (HPW == 2 && i == 1) {
                        h0[i] = wv & 1;
                        h1[i] = wv < 4 ? h0[i] + 1 : 0;
                    }
                    if (kt[i] >= NTILE) kt[i] = h1[i] = 0;           // none: any tile, not kept
                    mt[i] = kt[i] < 1 ? 0 : (kt[i] < 3 ? 1 : (kt[i] < 6 ? 2 : 3));
                    jt[i] = kt[i] - mt[i] * (mt[i] + 1) / 2;
                }
            }
            // the products of a wave's tiles side by side: each alone is a chain
#pragma unroll
            for (int i = 0; i < TPW; ++i) g[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (QN >= 2) {
#pragma unroll
                for (int u = 0; u < QN / 2; ++u) {
                    s16x4 b0[TPW], b1[TPW];
                    uint4 cc[TPW];
#pragma unroll
                    for (int i = 0; i < TPW; ++i) {
                        b0[i] = as_s16x4(sB[b_at<NS>(16 * jt[i] + col, 2 * u, grp)]);
                        b1[i] = as_s16x4(sB[b_at<NS>(16 * jt[i] + col, 2 * u + 1, grp)]);
                        if (!FULL || i == 0) cc[i] = sC[c_at<NS>(16 * mt[i] + col, 4 * u + grp)];
                        else cc[i] = cc[0];
                    }
#pragma unroll
                    for (int i = 0; i < TPW; ++i) g[i] = mma_k32(b0[i], b1[i], lo4(cc[i]), hi4(cc[i]), g[i]);
                }
            } else {
                const uint2 *c2 = reinterpret_cast<const uint2 *>(sC);
#pragma unroll
                for (int i = 0; i < TPW; ++i)
                    g[i] = mma_k16(as_s16x4(sB[b_at<NS>(16 * jt[i] + col, 0, grp)]),
                                   as_s16x4(c2[2 * c_at<NS>(16 * mt[i] + col, grp >> 1) + (grp & 1)]), g[i]);
            }
        }
        // ---- weights and split of the products above
        auto weigh = [&]() {
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const int t = 16 * mt[i] + col, j = 16 * jt[i] + 4 * grp;
#pragma unroll
                for (int h = 0; h < HPW; ++h) {
                    if (h < h0[i] || h >= h1[i]) continue;
                    const Decays &d = sD[h];
                    f32x4 m;
                    if (jt[i] != mt[i]) {
                        const bool below = !FULL || jt[i] < mt[i];
                        // E at the end of the tile between the two (one apart: no factor)
                        const float e = below ? (mt[i] > jt[i] + 1 ? d.Cs[16 * mt[i] - 1] - d.Cs[16 * jt[i] + 15] : 0.f)
                                              : (jt[i] > mt[i] + 1 ? d.Cs[16 * jt[i] - 1] - d.Cs[16 * mt[i] + 15] : 0.f);
                        const float f = (below ? d.La : d.Ua)[t] * ex2(e);
                        m = g[i] * (*reinterpret_cast<const f32x4 *>((below ? d.Lb : d.Ub) + j) * f);
                    } else {
                        const f32x4 cj = *reinterpret_cast<const f32x4 *>(&d.Cs[j]), dj = *reinterpret_cast<const f32x4 *>(&d.Dt[j]);
                        f32x4 ej = cj;
                        if constexpr (FULL) ej = *reinterpret_cast<const f32x4 *>(&d.Ex[j]);
                        const float ct = d.Cs[t], et = FULL ? d.Ex[t] : 0.f;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int jj = 4 * grp + r;
                            float w = ex2(FULL && jj > col ? ej[r] - et : ct - cj[r]);
                            if constexpr (FULL) w = jj == col ? 2.f : w;
                            m[r] = FULL || jj <= col ? g[i][r] * (w * dj[r]) : 0.f;
                        }
                    }
                    s16x4 mh, ml;
                    split4(m, mh, ml);
                    const uint2 h2 = as_u2(mh), l2 = as_u2(ml);
                    uint2 *dst = reinterpret_cast<uint2 *>(m_of(h)) + m_at(mt[i], jt[i]) + 2 * lane;
                    dst[0] = h2;
                    dst[128] = l2;
                }
            }
        };
        if constexpr (GRAM && !OVER) {
            if (a.y) weigh();
        }

        // ---- prefix term 2^{cs_t} (C_t . S) for this wave's columns (rows of the products: lane
        // (grp, col) holds columns 16 wave + 4 grp .. +3 of y at token 16 mt + col); the state is split into bf16
        // hi + lo a pair of tiles at a time
        f32x4 Y[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) Y[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (a.y) {
            if constexpr (QN >= 2) {
#pragma unroll
                for (int u = 0; u < QN / 2; ++u) {
                    uint4 cc[4];
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) cc[mt] = sC[c_at<NS>(16 * mt + col, 4 * u + grp)];
                    s16x4 h0, l0, h1, l1;
                    split4(S[2 * u], h0, l0);
                    split4(S[2 * u + 1], h1, l1);
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) Y[mt] = mma_k32(h0, h1, lo4(cc[mt]), hi4(cc[mt]), Y[mt]);
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) Y[mt] = mma_k32(l0, l1, lo4(cc[mt]), hi4(cc[mt]), Y[mt]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // (32-deep with a zero upper half: the products that follow add onto Y on that shape)
                const uint2 *c2 = reinterpret_cast<const uint2 *>(sC);
                constexpr s16x4 z = {0, 0, 0, 0};
                s16x4 h0, l0;
                split4(S[0], h0, l0);
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const s16x4 c0 = as_s16x4(c2[2 * c_at<NS>(16 * mt + col, grp >> 1) + (grp & 1)]);
                    Y[mt] = mma_k32(h0, z, c0, z, Y[mt]);
                    Y[mt] = mma_k32(l0, z, c0, z, Y[mt]);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) Y[mt] *= sEc[16 * mt + col];
        }
        if constexpr (GRAM && OVER) {
            __syncthreads();   // every wave has read C
            if (a.y) weigh();
        }
        if constexpr (GRAM) {
            __syncthreads();   // M published
            if (k + 1 < nch) st.issue(REV ? c - 1 : c + 1, tid, wave == 0);
        }

        if constexpr (!GRAM && HPW == 2) {
            if (k + 1 < nch) st.issue(REV ? c - 1 : c + 1, tid, wave == 0);
        }

        // x operands of this wave's columns (tokens 16jt + 4grp .. +3)
        s16x4 xh[4];
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) xh[jt] = x_read(sX, jt, wave, lane);
        if (a.y) {
            // ---- intra-chunk term: y += M x
            if constexpr (GRAM) {
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
                    for (int jt = 0; jt <= (FULL ? 3 : mt); jt += 2) {
                        const uint4 *mp = sM + m_at(mt, jt) / 2 + lane;
                        const uint4 mh = mp[0], ml = mp[64];
                        if (FULL || jt + 1 <= mt) {
                            Y[mt] = mma_k32(xh[jt], xh[jt + 1], lo4(mh), hi4(mh), Y[mt]);
                            Y[mt] = mma_k32(xh[jt], xh[jt + 1], lo4(ml), hi4(ml), Y[mt]);
                        } else {
                            // the accumulator comes from 32-deep MFMAs: stay on that shape (zero
                            // upper half) rather than hand it to a 16-deep MFMA
                            constexpr s16x4 z = {0, 0, 0, 0};
                            Y[mt] = mma_k32(xh[jt], z, lo4(mh), z, Y[mt]);
                            Y[mt] = mma_k32(xh[jt], z, lo4(ml), z, Y[mt]);
                        }
                    }
                }
            }
            // ---- skip term and store: the products are formed with the columns of y as rows, so a
            // lane holds four consecutive columns of one token and stores 16 bytes (as 4-byte
            // stores the passes that add spent over half of their wave cycles waiting to issue
            // them).  The four waves write a row's 256 bytes in 64-byte pieces at different
            // times: the passes that store do so through the cache, so the pieces meet in L2;
            // the passes that add read the line first, so their nontemporal stores find it there
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                f32x4 out = Y[mt];
                if constexpr (GRAM)
                    out += skip * quad_val(as_s16x4(reinterpret_cast<const uint2 *>(
                                      sX)[2 * x_at(16 * mt + col, 2 * wave + (grp >> 1)) + (grp & 1)]));
                if constexpr (REV) out += yv[mt];
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out), rY, y_off(mt), 0, REV ? kNT : 0);
            }
        }

        // ---- carry the state across the chunk (not after the last one unless it is kept)
        if (k + 1 == nch && !a.pool_out) break;
        const float keep = ex2(sCs[kC - 1]);
        WOps<T3> wx;
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
            w_set(wx, jt, *reinterpret_cast<const f32x4 *>(&sWs[16 * jt + 4 * grp]) * quad_val(xh[jt]));
        // tiles in pairs: the products of one tile are a chain, two run side by side
#pragma unroll
        for (int q = 0; q < QN; q += 2) {
            constexpr int D = QN >= 2 ? 2 : 1;
            s16x4 b[D][4];
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int jt = 0; jt < 4; ++jt) b[d][jt] = bt_read<NS>(sB, jt, q + d, lane);
#pragma unroll
            for (int d = 0; d < D; ++d) S[q + d] *= keep;
#pragma unroll
            for (int jt = 0; jt < 4; jt += 2) {
#pragma unroll
                for (int d = 0; d < D; ++d) S[q + d] = mma_k32(b[d][jt], b[d][jt + 1], wx.h[jt], wx.h[jt + 1], S[q + d]);
#pragma unroll
                for (int d = 0; d < D; ++d) S[q + d] = mma_k32(b[d][jt], b[d][jt + 1], wx.l[jt], wx.l[jt + 1], S[q + d]);
                if constexpr (T3) {
#pragma unroll
                    for (int d = 0; d < D; ++d) S[q + d] = mma_k32(b[d][jt], b[d][jt + 1], wx.m[jt], wx.m[jt + 1], S[q + d]);
                }
            }
        }
        __syncthreads();   // LDS is rewritten by the next chunk
    }
    if (a.pool_out) {
        float *dst = a.pool_out + (cslot * a.nheads + un.h) * (kP * NS);
#pragma unroll
        for (int q = 0; q < QN; ++q) *reinterpret_cast<f32x4 *>(dst + s_off(q)) = S[q];
    }
}

template <int NS, int HPW>
hipError_t out16(const SeqArgs &k, SeqOut what, unsigned grid, hipStream_t s) {
    const dim3 g(grid / HPW), b(kThreads * HPW);
    const bool kept = k.pool_out != nullptr;   // the carried state is written out
    if (what == SeqOut::kFwd) {
        if constexpr (HPW == 2) {
            if (kept) hipLaunchKernelGGL((bdlm_seg_out16_kernel<NS, 2, kFwd, true>), g, b, 0, s, k);
            else hipLaunchKernelGGL((bdlm_seg_out16_kernel<NS, 2, kFwd, false>), g, b, 0, s, k);
        } else {
            return hipErrorInvalidValue;       // (bdlm_seq.hip's kernel: seq16_forward)
        }
    } else if (kept) {
        hipLaunchKernelGGL((bdlm_seg_out16_kernel<NS, HPW, kBoth, true>), g, b, 0, s, k);
    } else {
        hipLaunchKernelGGL((bdlm_seg_out16_kernel<NS, HPW, kBoth, false>), g, b, 0, s, k);
    }
    return hipGetLastError();
}
template <int NS>
hipError_t out16_any(const SeqArgs &k, SeqOut what, unsigned grid, hipStream_t s) {
    if (what == SeqOut::kPre) {
        hipLaunchKernelGGL((bdlm_seg_out16_kernel<NS, 1, kPre, false>), dim3(grid), dim3(kThreads), 0, s, k);
        return hipGetLastError();
    }
    if (!seq16_pairs(k, grid)) return out16<NS, 1>(k, what, grid, s);
    SeqArgs p = k;
    p.xcd_remap = grid / 2 % 8 == 0 ? 1 : 0;
    return out16<NS, 2>(p, what, grid, s);
}
template <int NS>
hipError_t state16(const SeqArgs &k, bool both, unsigned grid, hipStream_t s) {
    if (both) hipLaunchKernelGGL((bdlm_seg_state16_kernel<NS, true>), dim3(grid), dim3(kThreads), 0, s, k);
    else hipLaunchKernelGGL((bdlm_seg_state16_kernel<NS, false>), dim3(grid), dim3(kThreads), 0, s, k);
    return hipGetLastError();
}
}  // namespace

// Two heads share a workgroup's B, C and C.B^T products where a group's heads pair up and the
// launch still fills the chip with half as many workgroups (two per CU: 512).  With fewer, more
// and smaller workgroups are faster: forward outputs of 640 row-heads 785 us against 799, of
// 896 280 against 268, of 4,096 1,147 against 1,093 (one segment, normalisation included).
bool seq16_pairs(const SeqArgs &k, unsigned grid) { return k.heads_per_group % 2 == 0 && grid >= 768; }
// Forward outputs in pairs of heads (else bdlm_seq.hip's kernel).  At dstate 32 and less three of
// the other's workgroups share a CU: pairs are faster only where they run in one round of two
// per CU and the others need a second.  Pairs over the others, one segment of 1,024 tokens,
// dstate 16 | 32: 768 row-heads 1.25 | 1.18, 896 0.90 | 0.86, 1,024 0.87 | 0.87, 1,280 1.09 |
// 1.11; several segments of 4,096 tokens, 288 row-heads 1.09 | 1.08 (dstate 64: 0.99, 128: 0.98).
bool seq16_forward(int ns, const SeqArgs &k, unsigned grid) {
    return seq16_pairs(k, grid) && (ns >= 64 || (k.nseg == 1 && grid > 768 && grid <= 1024));
}

hipError_t seq16_state(int ns, const SeqArgs &k, bool both, unsigned grid, hipStream_t s) {
    switch (ns) {
        case 16: return state16<16>(k, both, grid, s);
        case 32: return state16<32>(k, both, grid, s);
        case 64: return state16<64>(k, both, grid, s);
        case 128: return state16<128>(k, both, grid, s);
        default: return hipErrorInvalidValue;
    }
}
hipError_t seq16_out(int ns, const SeqArgs &k, SeqOut what, unsigned grid, hipStream_t s) {
    switch (ns) {
        case 16: return out16_any<16>(k, what, grid, s);
        case 32: return out16_any<32>(k, what, grid, s);
        case 64: return out16_any<64>(k, what, grid, s);
        case 128: return out16_any<128>(k, what, grid, s);
        default: return hipErrorInvalidValue;
    }
}
}  // namespace bdlm
