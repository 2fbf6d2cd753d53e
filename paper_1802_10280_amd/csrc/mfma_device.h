// Device code that the matrix-core kernels share: the arguments, and the way back to the nonzeros for outputs
// whose sums cannot be used.
#pragma once
#include "mfma.h"

namespace escoin {
namespace {

typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

struct MfmaArgs {
    const float* in;
    float* out;
    const float* bias;
    const b8* w;              // [32-row block][chunk of 16 channels][tap][split][lane]
    const int32_t* rowptr;    // the nonzeros once more, for sums that cannot be used
    const MfmaNz* nz;
    int N, C, H, W, M, E, F, R, S, pad, stride;
    int pitch, plane;         // of the flat padded array: columns per row, positions per image
    int n_chunks, n_mgroups, n_tiles;
    uint32_t flags;
};

constexpr float kTinyInput = 0x1p-70f, kTinySum = 0x1p-58f;

// An output's place: row and column of its first tap, and that tap's word in channel 0, counted from the first image
// that the workgroup touches (an offset from the batch's start would need 64 bits).
struct Place {
    int y, x, first;
};

// Every step-th nonzero from `j` on, for T positions of a lane.  Eight loads (sixteen for four positions) at a
// time and no branches, so that they are on their way together: past the end the last nonzero is read again,
// beside the image the first word of `input`, and neither counts.  Words: the nonzeros as MfmaNz is laid out; in the
// constant address space, where `j` is the same for the whole wave, they come through scalar loads.
template <int T, class Words>
__device__ inline void walk(const MfmaArgs& a, const float* input, Words nz, int j, int end, int step, const Place (&at)[T], float (&v)[T]) {
    constexpr int kBatch = T == 1 ? 8 : 4;
    const uint32_t* __restrict__ in = (const uint32_t*)input;
    for (; j < end; j += kBatch * step) {
        uint32_t c[kBatch], rs[kBatch], w[kBatch], keep[kBatch][T], x[kBatch][T];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const auto p = nz + 3 * min(j + b * step, end - 1);
            c[b] = p[0];
            rs[b] = p[1];
            w[b] = p[2];
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const int r = rs[b] & 0xffffu, s = rs[b] >> 16, off = ((int)c[b] * a.H + r) * a.W + s;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const bool inside = (uint32_t)(at[t].y + r) < (uint32_t)a.H & (uint32_t)(at[t].x + s) < (uint32_t)a.W & j + b * step < end;
                keep[b][t] = inside ? ~0u : 0u;
                x[b][t] = (off + at[t].first) & keep[b][t];
            }
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
#pragma unroll
            for (int t = 0; t < T; ++t) x[b][t] = in[x[b][t]];
        __builtin_amdgcn_sched_barrier(0);  // all on their way before the first is waited for
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
#pragma unroll
            for (int t = 0; t < T; ++t) v[t] = fmaf(__uint_as_float(w[b]), __uint_as_float(x[b][t] & keep[b][t]), v[t]);
    }
}
static_assert(sizeof(MfmaNz) == 12, "walk() reads three words a nonzero");

// The marked positions once more from the nonzeros, for the channels m0 .. m0 + rows - 1 of a workgroup whose
// `waves` waves share the channels; `only`: those with a bit there, where it is given.  `lists`: which of the RUNS * 64 positions from t0 on.
// Bound by the gathers' latency where few workgroups come here and by their address arithmetic where all
// do.  64x256x28x28 at 50 % in three bf16 parts, when each lane redid its own outputs -> now: one NaN in the batch 6.4 -> 0.5 ms,
// one image of them 11.6 -> 2.3, nothing else 32 -> 7.0 (the tiled kernel takes 0.72 whatever the input).  Pairs, whose
// workgroups have 64 positions, not 256, to a nonzero: 0.26, 2.3 and 16.0 (0.25 without any); two by 64 channels, at 80 %: 0.30, 1.6 and 6.4 (0.18).
template <int RUNS>
__device__ inline void redo(const MfmaArgs& a, const uint64_t (&lists)[RUNS], int t0, int m0, int rows, int waves, int wave, int lane,
                            const uint64_t* only = nullptr) {
    const bool relu = a.flags & ESCOIN_F_RELU, has_bias = a.flags & ESCOIN_F_BIAS;
    const int EF = a.E * a.F, HW = a.H * a.W, n_first = t0 / a.plane;
    const float* const in = a.in + (size_t)n_first * a.C * HW;
    const auto shared_nz = (const __attribute__((address_space(4))) uint32_t*)a.nz;
    int total = 0;
#pragma unroll
    for (int run = 0; run < RUNS; ++run) total += __popcll(lists[run]);
    const auto store = [&](float v, int m, int u) {
        const int n = u / a.plane, rem = u - n * a.plane, h = rem / a.pitch, x = rem % a.pitch;
        v += has_bias ? a.bias[m] : 0.0f;
        if (relu) v = v > 0.0f ? v : 0.0f;
        a.out[((size_t)n * a.M + m) * EF + h * a.F + x] = v;
    };
    const auto place = [&](int u) -> Place {
        const int n = u / a.plane, rem = u - n * a.plane, y = rem / a.pitch * a.stride - a.pad, x = rem % a.pitch * a.stride - a.pad;
        return {y, x, (n - n_first) * a.C * HW + y * a.W + x};
    };
    // More than half of them: a lane takes its position of every run at once, and a nonzero is read for all
    // (run by run those two last calls took 4.3 and 12.5 ms).
    if (total > RUNS * 32) {
        Place at[RUNS];
#pragma unroll
        for (int run = 0; run < RUNS; ++run) {
            at[run] = place(t0 + run * 64 + lane);
            if (!(lists[run] >> lane & 1)) at[run].y = -(1 << 30);  // no tap is inside
        }
        for (int k = wave; k < rows && m0 + k < a.M; k += waves) {
            const int m = m0 + k;
            if (only && !(only[k >> 6] >> (k & 63) & 1)) continue;
            float v[RUNS] = {};
            walk(a, in, shared_nz, __builtin_amdgcn_readfirstlane(a.rowptr[m]), __builtin_amdgcn_readfirstlane(a.rowptr[m + 1]), 1, at, v);
#pragma unroll
            for (int run = 0; run < RUNS; ++run)
                if (lists[run] >> lane & 1) store(v[run], m, t0 + run * 64 + lane);
        }
        return;
    }
    // Few: run by run, several lanes to an output's nonzeros where the run has 32 such positions or fewer.
    for (int run = 0; run < RUNS; ++run) {
        uint64_t list = lists[run];
        const int count = __popcll(list);
        if (count == 0) continue;
        const int shift = count > 1 ? __clz(count - 1) - 26 : 6;  // 64 >> shift is at least count
        const int mine = lane >> shift, step = 1 << shift, part = lane & (step - 1);
        const bool active = mine < count;  // the other lanes go along with the first position
        for (int k = 0; active && k < mine; ++k) list &= list - 1;
        const int u = t0 + run * 64 + __ffsll((unsigned long long)list) - 1;
        const Place at[1] = {place(u)};
        for (int k = wave; k < rows && m0 + k < a.M; k += waves) {
            if (only && !(only[k >> 6] >> (k & 63) & 1)) continue;
            const int m = m0 + k, begin = __builtin_amdgcn_readfirstlane(a.rowptr[m]), end = __builtin_amdgcn_readfirstlane(a.rowptr[m + 1]);
            float v[1] = {};
            if (step == 1) walk(a, in, shared_nz, begin, end, 1, at, v);
            else walk(a, in, (const uint32_t*)a.nz, begin + part, end, step, at, v);
            for (int s = 1; s < step; s <<= 1) v[0] += __shfl_xor(v[0], s);
            if (active && part == 0) store(v[0], m, u);
        }
    }
}

}  // namespace
}  // namespace escoin
