// sconv on the matrix cores for layers of fewer than 16 input channels and an even stride, as a network's first one: fp32 operands as pairs of
// fp16 numbers, as in sconv_pair.hip.
//
// With so few channels the 16 factors of a matrix instruction are not channels but neighbouring taps: half of them, 8, are
// 8 columns of one filter row of one channel (the last of them may be none: their weights are zero), so a 7x7 filter on 3 channels takes 12
// instructions to a product (21 groups of 8 columns in pairs, an even number of those) where 16 channels to a tap would take 49.  In LDS the input lies as it does in memory, padded, its two parts
// apart; a lane's 8 columns are 16 bytes of a row from its output's first column on, aligned to 4 bytes as the stride is even.
// A workgroup takes 64 channels of 256 consecutive outputs of an image, 32 a wave, and all input channels at once: its inputs pass
// through registers (24 words a lane, of whole padded rows: maps of 3 channels with 7x7 filters
// of stride 2 up to 250 columns wide, but for 123 to 126), so that the scale is that of the
// largest, and there is no second pass.  Two sums by turns halve the chains.
//
// Bound by its chain (inputs, barrier, largest, barrier, conversion, barrier, twelve steps whose weights are asked for one ahead, stores), as the
// matrix cores need 2 us.  32 positions a wave, not 64, so that two workgroups fit a compute unit without spills (288 registers; 31 us).
// 5x3x224x224, 64 7x7 filters of stride 2 at 50 %: 17.5 us, 29 with a channel too short for the pairs, the tiled
// kernel 41; 32 images 77 and 153.
#include <float.h>
#include <algorithm>

#include "common.h"
#include "mfma_device.h"
#include "pair.h"
#include "plan.h"

namespace escoin {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef int i4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef u4 u4_by_words __attribute__((aligned(4)));

struct FirstArgs : MfmaArgs {
    const int32_t* exps;  // of the rows' weights: what they were scaled up by
    int steps, width;     // steps of two groups of 8 columns; groups to a filter row
    int in_rows, columns; // of the padded input in LDS, a channel
    int few;              // channels with fewer nonzeros are computed from those
    int together;         // rows that the waves read at a time
    int n_tiles_image;
};

constexpr uint32_t kNowhere = 0x80000000u;  // past the end of the image
constexpr int kWaves = kFirstPositions / 32, kThreads = 64 * kWaves;

__global__ __launch_bounds__(kThreads, 4) void sconv_first_kernel(const FirstArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ uint64_t again[kWaves / 2];
    __shared__ uint32_t peak;
    __shared__ int lost;
    __shared__ uint32_t row_at[kFirstLoads * kWaves];  // a row's byte offset in the image
    __shared__ __attribute__((aligned(16))) int row_exp[64];
    __shared__ __attribute__((aligned(16))) float row_bias[64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int EF = a.E * a.F, HW = a.H * a.W;
    const int tile_at = blockIdx.x / a.n_mgroups, mg = blockIdx.x - tile_at * a.n_mgroups;
    const int image = tile_at / a.n_tiles_image, tile = tile_at - image * a.n_tiles_image;
    const int p0 = tile * kFirstPositions, h0 = p0 / a.F;
    const int words = a.C * a.in_rows * a.columns;
    _Float16* const high = (_Float16*)lds;
    _Float16* const low = high + words;
    int* const group_at = (int*)(low + words);  // and behind it room for what belongs nowhere
    const auto in = __builtin_amdgcn_make_buffer_rsrc((void*)(a.in + (size_t)image * a.C * HW), 0, a.C * HW * 4, 0x00020000);
    const bool relu = a.flags & ESCOIN_F_RELU, has_bias = a.flags & ESCOIN_F_BIAS;

    // ---- the input: a wave has 64 columns of every a.together-th row of the channels' rows
    const int n_rows = a.C * a.in_rows, runs = (a.columns + 63) / 64, mine = wave / runs;
    const int col = mine < a.together ? 64 * (wave - mine * runs) + lane : a.columns;  // of waves left over: none
    for (int i = tid; i < kFirstLoads * kWaves; i += kThreads) {
        const int c = i / a.in_rows, y = h0 * a.stride - a.pad + i - c * a.in_rows;
        row_at[i] = i < n_rows && (uint32_t)y < (uint32_t)a.H ? (uint32_t)(c * HW + y * a.W) * 4u : kNowhere;
    }
    __syncthreads();
    const u4* w = (const u4*)a.w + (size_t)mg * 2 * a.steps * 128 + lane;
    struct Weights { h8 p[2][2]; } w0, w1;  // of a step: 32 channels, part
    const auto weights = [&](Weights& o, int step) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < 2; ++k) o.p[p][k] = __builtin_bit_cast(h8, w[((size_t)p * a.steps + step) * 128 + k * 64]);
    };
    float x[kFirstLoads];
    const bool col_there = (uint32_t)(col - a.pad) < (uint32_t)a.W && col < a.columns;
#pragma unroll
    for (int b = 0; b < kFirstLoads; ++b) {
        const uint32_t row = row_at[(mine < a.together ? mine : 0) + b * a.together];
        x[b] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(in, col_there ? row + 4u * (col - a.pad) : kNowhere, 0, 0));
    }
    if (tid < 64) {
        row_exp[tid] = a.exps[min(mg * 64 + tid, a.M - 1)];
        row_bias[tid] = has_bias ? a.bias[min(mg * 64 + tid, a.M - 1)] : 0.0f;
    }
    if (tid < kWaves / 2) again[tid] = 0;
    if (tid == kWaves) peak = 0;
    if (tid == kWaves + 1) lost = 0;
    for (int g = tid; g < 2 * a.steps; g += kThreads) {
        const int row = g / a.width, j = g - row * a.width, c = row / a.R;
        group_at[g] = c < a.C ? (c * a.in_rows + row - c * a.R) * a.columns + 8 * j : 0;  // past the last weights are zero
    }
    __syncthreads();
    uint32_t most = 0;
#pragma unroll
    for (int b = 0; b < kFirstLoads; ++b) {
        const uint32_t u = __float_as_uint(x[b]) & 0x7fffffffu;
        most = max(most, u < 0x7f800000u ? +u : 0u);
    }
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) most = max(most, (uint32_t)__shfl_xor((int)most, s));
    if (lane == 0) atomicMax(&peak, most);
    __syncthreads();
    // Inputs are taken times 2^ex, the largest then below 2^15; those below 2^-13 lose bits.
    const uint32_t top_bits = __builtin_amdgcn_readfirstlane(peak);
    const int ex = (top_bits ? 127 - (int)(top_bits >> 23) : 0) + 14;
    const uint32_t least = (uint32_t)max(0, 127 - 13 - ex) << 23;
    int losing = 0;
    int at_row = mine * a.columns + col;
#pragma unroll
    for (int b = 0; b < kFirstLoads; ++b) {
        const bool there = col < a.columns && at_row < words;
        const _Float16 h = (_Float16)ldexpf(x[b], ex);
        high[there ? at_row : 2 * words + 4 * a.steps] = h;
        low[there ? at_row : words + 4 * a.steps] = (_Float16)fmaf(-2048.0f, (float)h, ldexpf(x[b], ex + 11));
        const uint32_t u = __float_as_uint(x[b]) & 0x7fffffffu;
        losing += u - 1u < least - 1u && least != 0 ? 1 : 0;
        at_row += a.together * a.columns;
    }
    if (losing) atomicAdd(&lost, losing);
    __syncthreads();

    // ---- products
    f16v big[2][2], small[2];  // sums of even and odd steps; 32 channels
#pragma unroll
    for (int p = 0; p < 2; ++p) { big[0][p] = (f16v)(0.0f); big[1][p] = (f16v)(0.0f); small[p] = (f16v)(0.0f); }
    int at = p0 + wave * 32 + (lane & 31);
    const int p = min(at, EF - 1), h = p / a.F, start = (h - h0) * a.stride * a.columns + (p - h * a.F) * a.stride;
    const int* const group = group_at + (lane >> 5);
    struct Inputs { h8 high, low; } x0, x1;
    const auto inputs = [&](Inputs& o, int step) {
        const int off = start + group[2 * step];
        o.high = __builtin_bit_cast(h8, *(const u4_by_words*)(high + off));
        o.low = __builtin_bit_cast(h8, *(const u4_by_words*)(low + off));
    };
    const auto step = [&](const Weights& c, const Inputs& x, f16v (&sum)[2]) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            sum[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c.p[p][0], x.high, sum[p], 0, 0, 0);
            small[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c.p[p][1], x.high, small[p], 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) small[p] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c.p[p][0], x.low, small[p], 0, 0, 0);
    };
    weights(w0, 0);
    inputs(x0, 0);
    for (int i = 0; i < a.steps; i += 2) {  // an even number of them
        weights(w1, i + 1);
        inputs(x1, i + 1);
        step(w0, x0, big[0]);
        const int ahead = min(i + 2, a.steps - 1);
        weights(w0, ahead);
        inputs(x0, ahead);
        step(w1, x1, big[1]);
    }

    // ---- a lane holds, per 32 channels, 16 channels of one position: 8*(i/4) + 4*(lane/32) + i%4
    const float small_sum = 2.0f * (float)lost;  // an input below 2^-13 is off by 2^-36 at most, a weight below 2^15
    const int m0 = mg * 64 + 4 * (lane >> 5), rows = a.M - m0;
    float* __restrict__ const o = a.out + ((size_t)image * a.M + m0) * EF + at;
    bool bad = false;
    if (at < EF) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int i = 0; i < 16; i += 4) {
                const int k0 = 32 * p + 2 * i;
                const i4 e = *(const i4*)(row_exp + 4 * (lane >> 5) + k0);
                const f4 b = *(const f4*)(row_bias + 4 * (lane >> 5) + k0);
                f4 y;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float v = fmaf(0x1p-11f, small[p][i + k], big[0][p][i + k] + big[1][p][i + k]);
                    bad |= k0 + k < rows && !(fabsf(v) <= FLT_MAX && fabsf(v) >= small_sum);
                    y[k] = ldexpf(v, -ex - e[k]) + b[k];
                    if (relu) y[k] = y[k] > 0.0f ? y[k] : 0.0f;
                }
                if (k0 + 4 <= rows) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) o[(size_t)(k0 + k) * EF] = y[k];
                } else {
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if (k0 + k < rows) o[(size_t)(k0 + k) * EF] = y[k];
                }
            }
    }
    const uint64_t lanes = __ballot(bad);
    if (lanes != 0 && lane == 0) atomicOr((unsigned long long*)&again[wave >> 1], ((lanes | lanes >> 32) & 0xffffffffu) << (32 * (wave & 1)));
    __syncthreads();  // and the stores before the ones of redo()
    uint64_t lists[kWaves / 2], any = 0;
#pragma unroll
    for (int run = 0; run < kWaves / 2; ++run) any |= lists[run] = again[run];
    if (__builtin_expect(any == 0 && a.few == 0, 1)) return;
    // Channels too short for pairs to be as exact as a chain of fp32 sums go through such a chain; the waves take them in turn (12 us for up
    // to eight; with half of the waves at a channel 7.5 for two).  (One call for both: inlined twice, 76 registers are spilled.)
    uint64_t list = 0;
    if (a.few != 0) {
        const int m = min(mg * 64 + lane, a.M - 1);
        list = __ballot(mg * 64 + lane < a.M && a.rowptr[m + 1] - a.rowptr[m] < a.few);
    }
    for (int turn = any != 0 ? -1 : 0; turn < 0 || list != 0; ++turn) {
        int from = mg * 64, count = 64, waves = kWaves, mine = wave;
        if (turn >= 0) {
            from += __ffsll((unsigned long long)list) - 1;
            list &= list - 1;
            if (turn % kWaves != wave) continue;
            count = waves = 1;
            mine = 0;
#pragma unroll
            for (int run = 0; run < kWaves / 2; ++run) lists[run] = __ballot(p0 + 64 * run + lane < EF);
        }
        redo(a, lists, image * EF + p0, from, count, waves, mine, lane);
        if (turn < 0) __syncthreads();  // those stores before a short channel's
    }
}

}  // namespace

int launch_sconv_first(const Dims& d, const PlanHeader& h, int few, const char* d_plan, const float* d_in, float* d_out, const float* d_bias,
                       uint32_t flags, hipStream_t stream) {
    FirstArgs a;
    const char* const section = d_plan + h.off_pair;
    a.in = d_in; a.out = d_out; a.bias = d_bias; a.flags = flags;
    a.w = (const b8*)section;
    a.exps = (const int32_t*)(section + pair_weight_bytes(d));
    a.rowptr = (const int32_t*)(d_plan + h.off_nz);
    a.nz = (const MfmaNz*)(d_plan + h.off_nz + mfma_rowptr_bytes(d));
    a.N = d.N; a.C = d.C; a.H = d.H; a.W = d.W; a.M = d.M; a.E = d.E; a.F = d.F; a.R = d.R; a.S = d.S; a.pad = d.pad; a.stride = d.stride;
    a.pitch = d.F;
    a.plane = d.E * d.F;
    a.n_mgroups = (d.M + 63) / 64;
    a.n_tiles_image = (a.plane + kFirstPositions - 1) / kFirstPositions;
    a.steps = first_steps(d);
    a.width = first_width(d);
    a.in_rows = first_in_rows(d);
    a.columns = first_columns(d);
    a.together = first_together(d);
    a.few = few;
    const int lds = first_lds_bytes(d);
    if (first_loads(d) > kFirstLoads) return ESCOIN_ERANGE;
    const unsigned blocks = (unsigned)(d.N * a.n_tiles_image * a.n_mgroups);
    return launch(sconv_first_kernel, dim3(blocks), dim3(kThreads), (size_t)lds, stream, a);
}

}  // namespace escoin
