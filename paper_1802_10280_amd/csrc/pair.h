// The layer on the matrix cores with fp32 operands as pairs of fp16 numbers: what its plan section holds and
// which layers have one.
#pragma once
#include "common.h"
#include "mfma.h"
#include "plan.h"

namespace escoin {

constexpr int kPairReach = 127;            // taps reach at most so many window positions past a workgroup's own
constexpr int kPairStepBytes = 2048;       // of 32 channels' weights for one tap of 16 input channels: two parts of 1024
constexpr int kPairLdsBytes = 160 * 1024;

// How a workgroup's waves are laid out: over 64 output channels each, 64 positions each, 16 input channels each.  Channels with
// fewer than `few` nonzeros are computed from those.  `flush`: after so many rounds a wave adds its sums to the workgroup's in LDS and
// starts again from zero, which makes the chains shorter and so more exact; 0: never.
struct PairShape {
    int MW, PW, KW, few = 0, flush = 0;
};
constexpr int kFewBatch = 16;              // that many of their nonzeros at a time
constexpr int kFewChains = 4;              // in so many chains of sums

// The flat padded map whose positions are numbered through the batch: columns a row, positions an image, and how far the taps
// reach.  At stride 1 the padding between rows and images is shared; at stride 2 the map is that of the outputs, a tap's inputs
// are those of one evenness of row and column (a phase: 2 * row + column), and each phase is a map of its own beside the others.
inline int pair_pitch(const Dims& d) { return d.stride == 2 ? d.F + (d.S - 1) / 2 : d.W + d.pad; }
inline long long pair_plane(const Dims& d) { return (long long)(d.stride == 2 ? d.E + (d.R - 1) / 2 : d.H + d.pad) * pair_pitch(d); }
inline long long pair_reach(const Dims& d) {
    return d.stride == 2 ? (long long)((d.R - 1) / 2) * pair_pitch(d) + (d.S - 1) / 2 : (long long)(d.R - 1) * pair_pitch(d) + d.S - 1;
}

// Stride 2: where a phase's positions start in the window; phase 4: where they end.  A phase reaches as far as its own taps.
inline int pair_phase_at(const Dims& d, const PairShape& s, int phase) {
    int at = 0;
    for (int k = 0; k < phase; ++k) {
        const int rows = d.R - 1 - k / 2, cols = d.S - 1 - k % 2;
        if (rows >= 0 && cols >= 0) at += 64 * s.PW + rows / 2 * pair_pitch(d) + cols / 2;
    }
    return at;
}
// window positions a channel takes in LDS
inline int pair_window(const Dims& d, const PairShape& s) {
    return (int)(((d.stride == 2 ? pair_phase_at(d, s, 4) : 64 * s.PW + pair_reach(d)) + 3) / 4 * 4);
}
// LDS: notes, the channels' exponents and biases, the positions' outputs and the window's words (head); then one
// window buffer, or two where there is more than one round of channels (stride 1); the waves' sums meet in the same place.  Behind them
// the workgroup's sums, where they are flushed.
inline int pair_head_bytes(const PairShape& s) { return 64 + 8 * 64 * s.MW + 4 * 64 * s.PW; }
inline int pair_lds_bytes(const Dims& d, const PairShape& s) {
    const int WR = pair_window(d, s), buffers = d.stride == 1 && (int)mfma_chunks(d) > s.KW ? 2 : 1;
    return pair_head_bytes(s) + 4 * WR + std::max(buffers * s.KW * 64 * WR, s.MW * s.PW * (s.KW - 1) * 64 * 256) + (s.flush ? s.MW * s.PW * 64 * 256 : 0);
}

// Layers of fewer channels than a chunk have a kernel of their own (sconv_first.hip), whose weights lie in groups of 8 columns of a filter row of a
// channel: groups to a filter row, and steps of two groups.  It takes tiles of the outputs of an image in their order; in LDS lie, for each channel, so many rows and
// columns of the padded input, in two parts, and where each group starts.
constexpr int kFirstPositions = 256, kFirstLoads = 24, kFirstSteps = 255;
inline bool first_layer(const Dims& d) { return d.C < 16; }
inline int first_width(const Dims& d) { return (d.S + 7) / 8; }
inline int first_steps(const Dims& d) { return (d.C * d.R * first_width(d) + 3) / 4 * 2; }  // an even number
inline int first_in_rows(const Dims& d) { return (std::min(d.E, (kFirstPositions - 2 + d.F) / d.F + 1) - 1) * d.stride + d.R; }
inline int first_columns(const Dims& d) { return (d.F - 1) * d.stride + 8 * first_width(d); }
inline int first_together(const Dims& d) { return 8 / ((first_columns(d) + 63) / 64); }  // rows that 8 waves of 64 columns read at a time
inline int first_loads(const Dims& d) { return first_together(d) ? (d.C * first_in_rows(d) + first_together(d) - 1) / first_together(d) : 1 << 30; }
// (its rows are kFirstLoads of eight waves' 64 columns at most)
static_assert(kFirstLoads * 8 * 64 * 4 + kFirstSteps * 8 + 4 <= 63 * 1024, "beside 1.3 KB of its own");
inline int first_lds_bytes(const Dims& d) { return d.C * first_in_rows(d) * first_columns(d) * 4 + first_steps(d) * 8 + 4; }

// two steps to ask for ahead
inline uint64_t pair_weight_bytes(const Dims& d) {
    if (first_layer(d)) return mfma_row_blocks(d) * first_steps(d) * kPairStepBytes;
    return (mfma_row_blocks(d) * mfma_chunks(d) * d.R * d.S + 2) * kPairStepBytes;
}
inline uint64_t pair_bytes(const Dims& d) { return pair_weight_bytes(d) + mfma_rowptr_bytes(d); }  // with the rows' exponents

// Where a wave's weights are, and where the next step's: a step is one tap of 16 input channels, a round's steps (chunk by chunk, tap
// by tap) are shared evenly by its KW waves, whole chunks where every wave has one.  A wave asks for two steps more than it
// has; those lie behind its last ones, never past the section.
#define ESCOIN_HD __host__ __device__ inline __attribute__((always_inline))
struct PairWalk {
    int KW, RS, n_chunks, n_rounds, block_bytes;  // block: 32 output channels
    int last_skip, last_more;                     // of the last round, which need not be whole
    int round, at, left;                          // at: byte offset of the first of the wave's two blocks

    ESCOIN_HD static int least(int a, int b) { return a < b ? a : b; }
    ESCOIN_HD int first_step(int r, int k) const { return least(KW, n_chunks - r * KW) * RS * k / KW; }
    // The first block of a wave: `mg` of the workgroups over the channels, wave `wm` of its MW; M: output channels.  A wave
    // past the last channel, of a workgroup that reaches over it, multiplies the last two blocks as well and stores nothing.
    ESCOIN_HD static int row_block(int mg, int MW, int wm, int M) { return least(mg * MW + wm, (M - 1) / 64) * 2; }
    ESCOIN_HD PairWalk(int kw, int rs, int chunks, int row_blk, int kg)
        : KW(kw), RS(rs), n_chunks(chunks), n_rounds((chunks + kw - 1) / kw), block_bytes(chunks * rs * kPairStepBytes) {
        const int regular_at = ((n_rounds - 1) * KW + kg) * RS * kPairStepBytes;  // of the last round, were it a whole one
        const int last_begin = first_step(n_rounds - 1, kg);
        last_skip = ((n_rounds - 1) * KW * RS + last_begin) * kPairStepBytes - regular_at;
        // three more than the last round has: what is asked for beyond its end does not turn to another round
        last_more = first_step(n_rounds - 1, kg + 1) - last_begin - RS + 3;
        const int only = n_rounds == 1 ? 1 : 0;
        round = 0;
        at = row_blk * block_bytes + kg * RS * kPairStepBytes + only * last_skip;
        left = RS + only * last_more;
    }
    ESCOIN_HD void next() {
        const int turn = --left <= 0 ? 1 : 0;
        round += turn;
        const int last = round >= n_rounds - 1 ? turn : 0;
        at += kPairStepBytes + turn * (KW - 1) * RS * kPairStepBytes + last * last_skip;
        left += turn * RS + last * last_more;
    }
};

bool pair_planned(const Dims& d, long long nnz, const PlanHeader& h);
bool pair_taken(const Dims& d, const PlanHeader& h, PairShape* shape);
void pair_note_rows(const Dims& d, const int32_t* rp, PlanHeader* h);
bool pair_write(const Dims& d, const int32_t* rp, const MfmaNz* nz, char* out);
int launch_sconv_first(const Dims& d, const PlanHeader& h, int few, const char* d_plan, const float* d_in, float* d_out, const float* d_bias,
                       uint32_t flags, hipStream_t stream);
int launch_sconv_pair(const Dims& d, const PlanHeader& h, const PairShape& shape, const char* d_plan, const float* d_in, float* d_out,
                      const float* d_bias, uint32_t flags, hipStream_t stream);

}  // namespace escoin
