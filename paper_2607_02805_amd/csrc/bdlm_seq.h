// bdlm_seq.h -- what the two sources of the sequence kernels share: the kernel arguments, and
// the launch interface of the bf16 kernels (bdlm_seq16.hip) used by bdlm_seq.hip.  Internal.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bdlm.h"

namespace bdlm {

struct SeqArgs {
    const void *x, *dt, *Bm, *Cm;
    const float *A, *skip;       // skip: D (forward) or D_rev (reverse)
    const float *skip2;          // kBoth: D_rev beside skip's D; else nullptr
    float *y;                    // seg_out: outputs; nullptr: none
    float *ws;                   // segment states [unit][seg][dirs][64 * N] (pool layout)
    float *tot;                  // segment log2-decays [unit][seg]
    int64_t xs_b, xs_t, xs_h;
    int64_t dts_b, dts_t;
    int64_t bcs_b, bcs_t, bcs_g;
    int64_t T, S;                // tokens in the sequence; tokens per segment
    int32_t nseg, dirs;
    int32_t nheads, heads_per_group;
    int32_t zero_init;           // seg_out: every segment starts from zero (ws unused)
    int32_t xcd_remap;           // grid % 8 == 0: keep a (row, segment)'s heads on one XCD
    int32_t blk_major;           // states of (row, head, segment) at slot (row * nseg + segment)
                                 // * nheads + head (a pool of per-block states); else
                                 // (row * nheads + head) * nseg + segment
    // seg_out with one segment per row (a block step or commit of any length):
    const float *pool_in;        // the entering state from the cache (slot per row)
    float *pool_out;             // the final state written back to the cache (in place)
    // seg_out, forward: chunks of cstride (<= 64) tokens, and the state entering every
    // chunk written to emit[(row * emit_blocks + block) * nheads + head] (block = the
    // chunk's index in the sequence; segments hold whole chunks)
    int32_t cstride;
    float *emit;
    int64_t emit_blocks;
    int32_t use_slots;
    int32_t slots[BDLM_MAX_SLOT_ROWS];
};


// What one output launch of the bf16 kernels of bdlm_seq16.hip computes.
enum class SeqOut {
    kFwd,    // the forward branch; stores y (only where seq16_forward)
    kBoth,   // the forward branch and the reverse branch's part within each chunk; stores y
    kPre,    // the reverse branch's part from later chunks, added onto y (after kBoth)
};
bool seq16_pairs(const SeqArgs &k, unsigned grid);
bool seq16_forward(int ns, const SeqArgs &k, unsigned grid);
hipError_t seq16_state(int ns, const SeqArgs &k, bool both, unsigned grid, hipStream_t s);
hipError_t seq16_out(int ns, const SeqArgs &k, SeqOut what, unsigned grid, hipStream_t s);

}  // namespace bdlm
