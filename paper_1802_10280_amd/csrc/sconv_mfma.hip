// sconv on the matrix cores, for filter banks pruned so little that multiplying the zeros too costs
// less than walking the nonzeros.
//
// The layer is one product per filter tap: out[m, p] += W[m, c, tap] * in[c, p + shift(tap)], with the
// output positions p of the WHOLE batch numbered through one flat padded array (the 1-D array of
// Section 3.1, the padding between neighbouring rows and images shared: pitch W + pad, H + pad rows),
// so that a workgroup takes any kTP consecutive positions and small maps waste no lanes.
//
// fp32 is kept by splitting every operand into three bf16 parts, x = h + m + l, each the rounded rest
// of the one before: 8 + 8 + 8 significant bits, so the split of an fp32 number is exact.  Six of
// the nine partial products are formed (hh, hm, mh, mm, hl, lh); the three left out are below 2^-24
// of |x*w|, about the rounding of one fp32 product.  hh has an accumulator of its own, so that the
// running sum is rounded once per 16 channels, the five small ones share another.  An output of a single
// product is off by at most 9.7e-8 of it (fp32: 6.0e-8; root mean square 2.6e-8 and 2.5e-8), a sum of some
// hundred by a third of what the tiled kernel's chain of roundings gives.
//
// A finite input whose h rounds to infinity, an Inf or a NaN would spread to outputs that only meet
// it under a zero weight; and where a product passes the largest float, so may its parts, with both
// signs.  Either way the two sums hold an Inf or a NaN: a position with a sum that is not finite is
// computed again, from the nonzeros alone.
//
// bf16 ends at 2^-133, so the parts of an input below 2^-110 lose bits, and those of a product below
// 2^-120 too.  Staging notes whether it met a nonzero |x| below 2^-70 (weights are 2^-50 at least); if so,
// sums below 2^-58 are computed again as well.  In the others, what such inputs lose (3 * 2^-134 * 2^30 a
// product, fewer than 2^18 products) is below 2^-25 of the sum.
//
// Per wave and (tap, 16 channels) 12 MFMAs of 32 clk stand against 6 LDS reads and 3 KB of weights from
// L1/L2, which all the position waves of a workgroup share.  The MFMAs are about half of a full
// round's time (two workgroups of 16 chunks and 9 taps: 92 of 168 us at 2.4 GHz); the rest goes to staging,
// barriers and first waits, and to the last round, which is rarely full.  The weights lie in the plan in the order the lanes read them.  Eight waves at 128 registers let two workgroups
// share a compute unit and hide each other's staging, up to windows of 384 positions (the 96 KB of LDS a
// longer one takes fit once).  64x256x28x28, 256 3x3 filters at 50 %: 324 us
// (the MFMAs alone 152 us at 2.4 GHz; the 844 workgroups fill 1.65 rounds of 512) against 720 us
// in the tiled kernel; 64x384x13x13, 384 filters at 65 %: 234 against 313 us.  Asking for a step's
// weights a whole step ahead and staging through buffer loads changed neither (318, 233 us).
#include <float.h>

#include "common.h"
#include "mfma_device.h"
#include "plan.h"

namespace escoin {
namespace {

constexpr int kThreads = 64 * kMfmaWM * kMfmaWP;
constexpr int kTM = 32 * kMfmaWM;

// WR: window positions held in LDS (kTP and the reach of the taps, see mfma_window).
template <int WR>
__global__ __launch_bounds__(kThreads, 4) void sconv_mfma_kernel(const MfmaArgs a) {
    extern __shared__ __attribute__((aligned(16))) b8 win[];  // [buffer][split][8-channel half][WR]
    constexpr int kBuf = 6 * WR;
    constexpr int kTasks = (2 * WR + kThreads - 1) / kThreads;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = wave % kMfmaWP, wm = wave / kMfmaWP;

    // Workgroup ids land on the XCDs in turn (id mod 8): each XCD gets a contiguous range of the
    // tile-major order, so the channel groups of one tile read its input through one L2.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int jobs = a.n_tiles * a.n_mgroups, jq = jobs >> 3, jr = jobs & 7;
    if (slot >= jq + (xcd < jr ? 1 : 0)) return;  // the whole workgroup, before any barrier
    const int job = xcd * jq + min(xcd, jr) + slot;
    const int tile = job / a.n_mgroups, mg = job - tile * a.n_mgroups;
    const int t0 = tile * kMfmaTP;
    const int HW = a.H * a.W;

    // ---- staging: a task is one window position and 8 channels; which half is wave-uniform
    // because WR is a multiple of 64
    int src[kTasks];
#pragma unroll
    for (int i = 0; i < kTasks; ++i) {
        const int task = tid + i * kThreads;
        const int u = t0 + (task >= WR ? task - WR : task);
        const int n = u / a.plane, rem = u - n * a.plane;
        const int y = rem / a.pitch - a.pad, x = rem % a.pitch - a.pad;
        src[i] = (task < 2 * WR && n < a.N && y >= 0 && x >= 0) ? n * a.C * HW + y * a.W + x : -1;
    }
    float st[kTasks][8];
    auto fetch = [&](int kc) {
#pragma unroll
        for (int i = 0; i < kTasks; ++i) {
            const int half = (wave * 64 + i * kThreads) >= WR ? 1 : 0;  // wave-uniform
            const int c0 = kc * 16 + half * 8;
            const float* __restrict__ p = a.in + (size_t)c0 * HW;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                st[i][j] = 0.0f;
                if (c0 + j < a.C && src[i] >= 0) st[i][j] = p[(size_t)j * HW + src[i]];
            }
        }
    };
    uint32_t least = 0xffffffffu;  // of the nonzero |x|, as 2 * bits - 1 (a zero becomes the largest)
    auto commit = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kTasks; ++i) {
            const int task = tid + i * kThreads;
            b8 h, m, l;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float x = st[i][j];
                least = min(least, (__float_as_uint(x) << 1) - 1u);
                h[j] = (__bf16)x;
                const float r = x - (float)h[j];
                m[j] = (__bf16)r;
                l[j] = (__bf16)(r - (float)m[j]);
            }
            if (2 * WR % kThreads == 0 || task < 2 * WR) {
                b8* const o = win + buf * kBuf + task;
                o[0] = h;
                o[2 * WR] = m;
                o[4 * WR] = l;
            }
        }
    };

    f16v big[2], small[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) { big[q] = (f16v)(0.0f); small[q] = (f16v)(0.0f); }

    const int RS = a.R * a.S;
    const int row_blk = mg * kMfmaWM + wm;
    const b8* __restrict__ w = a.w + (size_t)row_blk * a.n_chunks * RS * 192 + lane;
    b8 wa[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) wa[s] = w[64 * s];
    fetch(0);
    commit(0);
    __syncthreads();
    // what the waves tell each other at the end, in the buffer the last chunk leaves free
    struct Notes { uint32_t tiny[kMfmaWM * kMfmaWP]; uint64_t again[kMfmaWM * kMfmaWP]; };
    Notes* const notes = (Notes*)(win + (a.n_chunks & 1) * kBuf);
    for (int kc = 0; kc < a.n_chunks; ++kc) {
        const bool more = kc + 1 < a.n_chunks;
        if (more) fetch(kc + 1);
        const b8* row = win + (kc & 1) * kBuf + (lane >> 5) * WR + wp * 64 + (lane & 31);
        for (int r = 0; r < a.R; ++r, row += a.pitch - a.S)
#pragma unroll 1
            for (int s = 0; s < a.S; ++s, ++row) {
                b8 x[2][3];
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int k = 0; k < 3; ++k) x[q][k] = row[32 * q + 2 * WR * k];
                const b8 c0 = wa[0], c1 = wa[1], c2 = wa[2];
                w += 192;  // the table ends with one spare step
#pragma unroll
                for (int k = 0; k < 3; ++k) wa[k] = w[64 * k];
#define ESCOIN_MFMA(ACC, A, B)                                                                            \
    _Pragma("unroll") for (int q = 0; q < 2; ++q) ACC[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, x[q][B], ACC[q], 0, 0, 0);
                ESCOIN_MFMA(big, c0, 0)
                ESCOIN_MFMA(small, c2, 0)
                ESCOIN_MFMA(small, c0, 2)
                ESCOIN_MFMA(small, c1, 1)
                ESCOIN_MFMA(small, c1, 0)
                ESCOIN_MFMA(small, c0, 1)
#undef ESCOIN_MFMA
            }
        // the other buffer was last read before the previous barrier
        if (more) {
            commit((kc + 1) & 1);
        } else {
            const bool met = __any(least < 2u * __float_as_uint(kTinyInput) - 1u);
            if (lane == 0) notes->tiny[wave] = met;
        }
        __syncthreads();
    }

    uint32_t tiny = 0;
#pragma unroll
    for (int k = 0; k < kMfmaWM * kMfmaWP; ++k) tiny |= notes->tiny[k];
    const bool relu = a.flags & ESCOIN_F_RELU, has_bias = a.flags & ESCOIN_F_BIAS;
    const int EF = a.E * a.F;
    // A lane holds, per 32 positions, 16 output channels of one position: 8*(i/4) + 4*(lane/32) + i%4.
    uint64_t again = 0;  // the wave's positions that have a sum that cannot be used
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int u = t0 + wp * 64 + q * 32 + (lane & 31);
        const int n = u / a.plane, rem = u - n * a.plane, h = rem / a.pitch, x = rem % a.pitch;
        const int m0 = row_blk * 32 + 4 * (lane >> 5);
        bool bad = false;
        if (n < a.N && h < a.E && x < a.F) {
            float* __restrict__ o = a.out + ((size_t)n * a.M + m0) * EF + h * a.F + x;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int dm = 8 * (i / 4) + i % 4;
                if (m0 + dm >= a.M) continue;
                const float sum = big[q][i] + small[q][i];
                bad |= !(fabsf(sum) <= FLT_MAX) || (tiny && fabsf(sum) < kTinySum);
                float v = sum + (has_bias ? a.bias[m0 + dm] : 0.0f);
                if (relu) v = v > 0.0f ? v : 0.0f;
                o[(size_t)dm * EF] = v;
            }
        }
        const uint64_t lanes = __ballot(bad);
        again |= ((lanes | lanes >> 32) & 0xffffffffu) << (32 * q);
    }
    if (lane == 0) notes->again[wave] = again;
    __syncthreads();
    uint64_t any = 0;
#pragma unroll
    for (int k = 0; k < kMfmaWM * kMfmaWP; ++k) any |= notes->again[k];
    if (any == 0) return;

    // Those positions once more from the nonzeros, all channels of the workgroup: its waves share the
    // channels.  (A position of one wave belongs to the waves of the other channels as well, so the lists meet
    // in LDS; the barrier also orders these stores after the ones above.)
    uint64_t lists[kMfmaWP];
#pragma unroll
    for (int run = 0; run < kMfmaWP; ++run) {
        lists[run] = 0;
#pragma unroll
        for (int k = 0; k < kMfmaWM; ++k) lists[run] |= notes->again[k * kMfmaWP + run];
    }
    redo(a, lists, t0, mg * kTM, kTM, kMfmaWM * kMfmaWP, wave, lane);
}

template <int WR>
int start(const MfmaArgs& a, unsigned blocks, hipStream_t stream) {
    // Two workgroups fit a compute unit (one, with the longest windows) and share its matrix cores.  A launch
    // that has no more than one for each compute unit asks for so much LDS that they do not double up
    // beside idle ones.
    constexpr int two = 2 * 6 * WR * 16;
    static_assert((2 * two <= 160 * 1024) == (WR <= kMfmaPairWindow), "the rule counts on this");
    const int lds = blocks <= 256 ? std::max(two, 84 * 1024) : two;
    if (lds > 64 * 1024) {
        const int rc = allow_dynamic_lds((const void*)sconv_mfma_kernel<WR>, lds);
        if (rc != ESCOIN_OK) return rc;
    }
    return launch(sconv_mfma_kernel<WR>, dim3(blocks), dim3(kThreads), (size_t)lds, stream, a);
}

}  // namespace

int launch_sconv_mfma(const Dims& d, const PlanHeader& h, const char* d_plan, const float* d_in, float* d_out,
                      const float* d_bias, uint32_t flags, hipStream_t stream) {
    MfmaArgs a;
    a.in = d_in; a.out = d_out; a.bias = d_bias; a.flags = flags;
    a.w = (const b8*)(d_plan + h.off_mfma);
    a.rowptr = (const int32_t*)(d_plan + h.off_mfma + mfma_weight_bytes(d));
    a.nz = (const MfmaNz*)(d_plan + h.off_mfma + mfma_weight_bytes(d) + mfma_rowptr_bytes(d));
    a.N = d.N; a.C = d.C; a.H = d.H; a.W = d.W; a.M = d.M; a.E = d.E; a.F = d.F; a.R = d.R; a.S = d.S; a.pad = d.pad; a.stride = d.stride;
    a.pitch = d.W + d.pad;
    a.plane = (d.H + d.pad) * a.pitch;
    a.n_chunks = (d.C + 15) / 16;
    a.n_mgroups = (d.M + kTM - 1) / kTM;
    a.n_tiles = (d.N * a.plane + kMfmaTP - 1) / kMfmaTP;
    const unsigned blocks = (unsigned)((long long)a.n_tiles * a.n_mgroups + 7) / 8 * 8;
    const int window = mfma_window(d);
    if (window <= 320) return start<320>(a, blocks, stream);
    if (window <= kMfmaPairWindow) return start<kMfmaPairWindow>(a, blocks, stream);
    return start<512>(a, blocks, stream);
}

}  // namespace escoin
