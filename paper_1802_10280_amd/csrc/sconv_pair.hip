// sconv on the matrix cores with fp32 operands as pairs of fp16 numbers, for all but the most heavily pruned layers of
// stride 1 and 2.
//
// The layer is one product per filter tap over the flat padded positions of the whole batch, zeros included, as in
// sconv_mfma.hip.  There an operand is three bf16 parts and a product six matrix instructions, here two fp16
// parts and three:
//   x = h + l / 2^11,  h = fp16(x), l = fp16((x - h) * 2^11),   x*w = hh + (hl + lh) / 2^11.
// (A published method: Ootomo and Yokota, "Recovering single precision accuracy from Tensor Cores while surpassing the FP32
// theoretical peak performance", 2022.)  h and l hold 22 bits and l's sign; l is scaled so that its exponent ends where h's does.  The product left out and the bits
// lost make a product uncertain by 2^-21 at most, 0.7e-7 in the mean: more than one fp32 rounding, less than a chain of
// some fifty.  hh has an accumulator of its own, and the channels are shared by several waves, whose sums meet at the end: the
// shorter chains are more exact (the rule in pair_plan.cpp weighs the forms' errors).
//
// fp16 ends at 2^16 and 2^-24, so inputs are scaled by a power of two, one for a workgroup: the first 32 channels or so that it
// stages are put below 2^10, later ones have 2^6 of room.  If a sum is not finite in the end, the workgroup looks for
// its largest finite input and goes through its channels again with the scale for that one; what is not finite then
// met an Inf, a NaN or a sum past fp32, and is computed from the nonzeros (redo()).  Inputs below 2^-13, scaled, lose bits:
// their number bounds what a sum may have lost, and sums too small for that go the same way.
//
// A wave takes 64 channels by 64 positions of one chunk of 16 input channels at a time: 12 matrix instructions of 32 clocks a
// tap against four 16-byte LDS reads and 4 KB of weights from L1/L2, asked for two taps ahead.  One wave alone issues
// too slowly to keep a matrix core busy (a tap took 1100 clocks where what lies around its instructions was in one
// place): the rest of a step is strung out between them and, for filters three wide, a row of taps is one block without
// address arithmetic.  Staging the next chunks goes along in the same way.
//
// At stride 2 the positions are the outputs', and a tap reads one of four phases of the input (rows and columns of one evenness),
// all of which a round stages side by side: the window is four times as large beside the same steps, so it has one buffer and two
// workgroups to a compute unit hide each other's staging (phase after phase, as rounds of their own: no faster than the tiled kernel).
// 32x128x56x56, 128 3x3 filters, 80 %: 38 us (tiled 70); 11x78x45x45, 439 5x5 filters, 71 %: 50 (125); 13x89x23x23, 276 3x3, 71 %: 17.5 (24).
// Measured: 64x256x28x28, 256 3x3 filters: 149-154 us at 80 % (tiled kernel 312), at 50 % 169-175 (323); 64x384x13x13, 384 filters, 65 %: 105-107 (three
// bf16 parts: 232); 32x64x56x56 at 80 %: 33.5 (48); 32x512x7x7 at 80 %: 30 (58).  The matrix cores are busy half of the time in the first
// one (76 us at 2.4 GHz) and a third where eight waves share the channels (counters, first call after others); the rest is the workgroups'
// beginnings and ends, 12000-17000 clocks each, which only the other workgroup of a compute unit hides (there is none beside eight
// waves), and the first two rounds, when all of them ask for their inputs at once.  Scalar registers are spilled (38 to 80),
// one or two of them read back in the loops over the steps.
#include <float.h>
#include <algorithm>

#include "common.h"
#include "mfma_device.h"
#include "pair.h"
#include "plan.h"

namespace escoin {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef int i4 __attribute__((ext_vector_type(4)));

// Loads through a buffer descriptor: what lies past its end reads as zero, and the scalar offset costs no vector
// instruction.
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ inline Rsrc rsrc_of(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}
constexpr uint32_t kNowhere = 0x80000000u;  // past the end of every descriptor here

struct PairArgs : MfmaArgs {
    const int32_t* exps;      // of the rows' weights: what they were scaled up by
    int WR;          // window positions a channel takes in LDS
    int groups;      // of 64 window positions
    uint32_t w_bytes;
    int few;         // channels with fewer nonzeros are computed from those
    int total_at;    // of the flushed sums, behind the window
    int flush;       // rounds between a wave's flushes, 0: none
    int phase_at[4]; // stride 2: where the window's rows and columns of each evenness (2 * row + column) start, in positions
};

#define ESCOIN_INLINE __attribute__((always_inline))
constexpr int kStepBytes = kPairStepBytes;
constexpr int kFewBad = 8;  // positions

// x / d and what is left, for x and d below 2^22 (one_over: 1 / d, rounded): the product is off by less than one.
__device__ inline int divide(int x, int d, float one_over, int* rest) {
    int q = (int)((float)x * one_over), r = x - q * d;
    if (r < 0) { --q; r += d; }
    if (r >= d) { ++q; r -= d; }
    *rest = r;
    return q;
}

// The largest of the wave's values, in lane 63: lane shifts of 1, 2, 4, 8 in rows of 16, then the rows' last lanes.
__device__ inline uint32_t wave_max(uint32_t x) {
#define ESCOIN_DPP(CTRL, ROWS) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false));
    ESCOIN_DPP(0x111, 0xf) ESCOIN_DPP(0x112, 0xf) ESCOIN_DPP(0x114, 0xf) ESCOIN_DPP(0x118, 0xf) ESCOIN_DPP(0x142, 0xa) ESCOIN_DPP(0x143, 0xc)
#undef ESCOIN_DPP
    return x;
}

// What the waves of a workgroup tell each other.
template <int PW>
struct Notes {
    uint64_t again[PW];  // positions that have a sum that cannot be used
    uint64_t rows[2];    // channels that have one
    int over;            // not 0: one of them is not finite
    int lost;            // eights of inputs with one that loses bits, zeros apart
    uint32_t peak;       // bits of the largest finite |x| that the scale is made for
};

// The LDS of a workgroup.
template <int MW, int PW>
struct Room {
    static constexpr int kHead = 64 + 8 * 64 * MW + 4 * 64 * PW;  // pair_head_bytes()
    char* lds;
    int WR;
    __device__ Notes<PW>* notes() const { return (Notes<PW>*)lds; }
    __device__ int* row_exp() const { return (int*)(lds + 64); }
    __device__ float* row_bias() const { return (float*)(lds + 64 + 4 * 64 * MW); }
    // offset of a position's output, channel 0 of image n_first being 0; -1 where it is none
    __device__ int* out_at() const { return (int*)(lds + 64 + 8 * 64 * MW); }
    __device__ uint32_t* tab() const { return (uint32_t*)(lds + kHead); }  // [WR]: byte offset of a window position in channel 0
    __device__ char* win() const { return lds + kHead + 4 * WR; }          // [buffer][chunk of the round][part][8-channel half][WR] x 16 bytes
};

// One pass over all channels: the wave's share of the sums, scaled by 2^-(ex + the row's exponent) in `v`, and which
// positions have one that cannot be used.  FLUSH: with the sums flushed now and then (PairShape).  STRIDE 2: on
// the window's four phases, in one buffer (pair.h).  AGAIN: with the scale for notes.peak, not one guessed from the first inputs.
template <int MW, int PW, int KW, bool FLUSH, int STRIDE, bool AGAIN>
__device__ __forceinline__ uint64_t pass(const PairArgs& a, const Room<MW, PW> room, Rsrc in, Rsrc wr, int lane, int wave, int mg, float (&v)[64 / KW],
                                         int* scale) {
    constexpr int kWaves = MW * PW * KW, TM = 64 * MW;
    const int wp = wave % PW, kg = wave / PW % KW, wm = wave / (PW * KW);
    const int WR = room.WR, sub_bytes = 4 * 16 * WR, buf_bytes = KW * sub_bytes;
    char* const win = room.win();
    const uint32_t* const tab = room.tab();
    f4* const total = (f4*)(win + a.total_at) + (wm * PW + wp) * 16 * 64 + lane;  // as `big` lies, four values at a time
    Notes<PW>* const notes = room.notes();
    const int HW4 = a.H * a.W * 4, last_channel = (a.C - 1) * HW4, RS = a.R * a.S;
    // What the steps ask for runs two steps ahead of them, through the rounds.
    PairWalk ask(KW, RS, a.n_chunks, PairWalk::row_block(mg, MW, wm, a.M), kg);
    const int n_rounds = ask.n_rounds;

    // ---- staging: a task is one 8-channel half of a chunk and 64 window positions (the last 64 overlap the ones
    // before); one past the last stands for the last, so that every wave has the same number of them.  Channels past
    // the end repeat the last one: their weights are zero.
    const int n_tasks = 2 * KW * a.groups, my_tasks = (n_tasks + kWaves - 1) / kWaves, in_threes = my_tasks / 3 * 3;
    struct Task { float x[8]; uint32_t src; int half, first; };
    auto locate = [&](Task& t, int index) ESCOIN_INLINE {
        const int task = min(wave + index * kWaves, n_tasks - 1);
        t.half = task & (2 * KW - 1);
        t.first = min(task / (2 * KW) * 64, WR - 64);
        t.src = tab[t.first + lane];
    };
    auto fetch_four = [&](Task& t, int round, auto first) ESCOIN_INLINE {
        constexpr int kFirst = decltype(first)::value;
        const int from = (round * KW * 2 + t.half) * 8 * HW4;
#pragma unroll
        for (int j = kFirst; j < kFirst + 4; ++j)
            t.x[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(in, t.src, min(from + j * HW4, last_channel), 0));
    };
    typedef std::integral_constant<int, 0> First;
    typedef std::integral_constant<int, 4> Second;
    auto fetch = [&](Task& t, int round) ESCOIN_INLINE {
        fetch_four(t, round, First{});
        fetch_four(t, round, Second{});
    };
    int ex = 0;         // inputs are taken times 2^ex
    uint32_t low = 0;   // twice the bits of the least |x| of which that loses nothing
    int lost = 0;
    auto commit = [&](const Task& t, int buf) ESCOIN_INLINE {
        h8 h, l;
        uint32_t least = 0xffffffffu;  // as 2 * bits - 1: a zero becomes the largest
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            const float2v x = {ldexpf(t.x[j], ex), ldexpf(t.x[j + 1], ex)};
            const h2 hh = __builtin_convertvector(x, h2);
            h[j] = hh[0];
            h[j + 1] = hh[1];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                least = min(least, (__float_as_uint(t.x[j + k]) << 1) - 1u);
                l[j + k] = (_Float16)fmaf(-2048.0f, (float)hh[k], ldexpf(t.x[j + k], ex + 11));
            }
        }
        lost += least < low ? 1 : 0;
        h8* const o = (h8*)(win + buf * buf_bytes + (t.half >> 1) * sub_bytes) + (t.half & 1) * WR + t.first + lane;
        o[0] = h;
        o[2 * WR] = l;
    };

    const auto tap_at = [&](int r, int s) ESCOIN_INLINE -> int {
        if (STRIDE == 1) return r * a.pitch + s;
        const int even = s & 1 ? a.phase_at[1] : a.phase_at[0], odd = s & 1 ? a.phase_at[3] : a.phase_at[2];
        return (r & 1 ? odd : even) + (r >> 1) * a.pitch + (s >> 1);
    };

    f16v big[2][2], small[2][2];
    struct Weights { u4 p[2][2]; } w0, w1, w2;
    auto weights = [&](Weights& o, int k, int p, int further = 0) ESCOIN_INLINE {
        o.p[p][k] = __builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16 + k * 1024 + further, p ? ask.at + ask.block_bytes : ask.at, 0);
    };
    auto all_weights = [&](Weights& o) ESCOIN_INLINE {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int p = 0; p < 2; ++p) weights(o, k, p);
        ask.next();
    };

    // Every round but the last gives each wave RS steps, so none is empty before the last; there, a wave without
    // steps only helps with the staging.
    Task ta, tb, tc;
    const bool three_ahead = STRIDE == 2 || a.S != 3;  // of the next round's tasks; filters three wide ask for them on the way
    {
        Task t[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) locate(t[k], k);
#pragma unroll
        for (int k = 0; k < 4; ++k) fetch(t[k], 0);
        if (my_tasks > 4) {
#pragma unroll
            for (int k = 4; k < 8; ++k) locate(t[k], k);
#pragma unroll
            for (int k = 4; k < 8; ++k) fetch(t[k], 0);
        }
        all_weights(w0);
        all_weights(w1);
        if (!AGAIN) {
            uint32_t most = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t b = __float_as_uint(t[k].x[j]) & 0x7fffffffu;
                    most = max(most, b < 0x7f800000u ? +b : 0u);
                }
            most = wave_max(most);
            if (lane == 63) atomicMax(&notes->peak, most);
        }
        __syncthreads();
        const uint32_t peak = __builtin_amdgcn_readfirstlane(notes->peak);
        // 2^6 of room above the first ones, where the second pass knows the largest
        ex = (peak ? 127 - (int)(peak >> 23) : 0) + (AGAIN ? 14 : 9);
        low = (uint32_t)max(0, 127 - 13 - ex) << 24;
#pragma unroll
        for (int k = 0; k < 4; ++k) commit(t[k], 0);
        if (my_tasks > 4) {
#pragma unroll
            for (int k = 4; k < 8; ++k) commit(t[k], 0);
        }
        for (int i = 8; i < my_tasks; ++i) {
            locate(ta, i);
            fetch(ta, 0);
            commit(ta, 0);
        }
    }
    locate(ta, 0);
    locate(tb, 1);
    locate(tc, 2);
    if (n_rounds > 1) {
        fetch(ta, 1);
        fetch(tb, 1);
        if (three_ahead) fetch(tc, 1);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) { big[p][q] = (f16v)(0.0f); small[p][q] = (f16v)(0.0f); }
    __syncthreads();
    for (int round = 0; round < n_rounds; ++round) {
        const bool more = round + 1 < n_rounds;
        const int buf = STRIDE == 2 ? 0 : round & 1, other = STRIDE == 2 ? 0 : buf ^ 1;
        const int begin = ask.first_step(round, kg), end = ask.first_step(round, kg + 1);
        int sub = begin / RS, tap = begin - sub * RS, r = tap / a.S, s = tap - r * a.S;
        const char* base = win + buf * buf_bytes + sub * sub_bytes + ((lane >> 5) * WR + wp * 64 + (lane & 31)) * 16;
        const char* row = base + tap_at(r, s) * 16;
        h8 xh0, xh1;
        const auto read = [&](int k, int q) ESCOIN_INLINE -> h8 { return *(const h8*)(row + (32 * q + 2 * WR * k) * 16); };
        int i = begin, task = 0;
        auto step = [&](const Weights& c, Weights& cn) ESCOIN_INLINE {
            __builtin_amdgcn_s_waitcnt(0x0f74);  // the step's weights were asked for two steps ago, the next one's are younger
            // One wave issues too slowly to keep the matrix cores busy with what a step needs around them in one
            // place: a little of it follows each matrix instruction.
#define ESCOIN_FENCE __builtin_amdgcn_sched_barrier(0x6);
#define ESCOIN_MFMA(ACC, A, B, P, Q)                                                                                    \
    ESCOIN_FENCE                                                                                                        \
    ACC[P][Q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, c.p[P][A]), B##Q, ACC[P][Q], 0, 0, 0); \
    ESCOIN_FENCE
            h8 xl0, xl1;
            ESCOIN_MFMA(big, 0, xh, 0, 0)
            xl0 = read(1, 0);
            ESCOIN_MFMA(big, 0, xh, 0, 1)
            xl1 = read(1, 1);
            row += 16;
            if (++s == a.S) {
                s = 0;
                row += (a.pitch - a.S) * 16;
                if (++r == a.R) {
                    r = 0;
                    row += sub_bytes - a.R * a.pitch * 16;
                    base += sub_bytes;
                }
            }
            if (STRIDE == 2) row = base + tap_at(r, s) * 16;
            ESCOIN_MFMA(big, 0, xh, 1, 0)
            ESCOIN_MFMA(big, 0, xh, 1, 1)
            ESCOIN_MFMA(small, 1, xh, 0, 0)
            weights(cn, 0, 0);
            ESCOIN_MFMA(small, 1, xh, 0, 1)
            weights(cn, 0, 1);
            ESCOIN_MFMA(small, 1, xh, 1, 0)
            weights(cn, 1, 0);
            ESCOIN_MFMA(small, 1, xh, 1, 1)
            weights(cn, 1, 1);
            ask.next();
            xh0 = read(0, 0);  // the next step's; after the last one what lies behind is read and not used
            xh1 = read(0, 1);
            __builtin_amdgcn_sched_barrier(0);  // a task is not looked at before this
            ESCOIN_MFMA(small, 0, xl, 0, 0)
            ESCOIN_MFMA(small, 0, xl, 0, 1)
            ESCOIN_MFMA(small, 0, xl, 1, 0)
            ESCOIN_MFMA(small, 0, xl, 1, 1)
            ESCOIN_FENCE
#undef ESCOIN_MFMA
#undef ESCOIN_FENCE
            ++i;
        };
        // The three taps of a filter row at a time, where the filter is three wide: no addresses to work out between.
        const int part = 2 * WR * 16;
        auto three = [&](auto stage) ESCOIN_INLINE {
            constexpr bool STAGE = decltype(stage)::value;
#define ESCOIN_FENCE __builtin_amdgcn_sched_barrier(0x6);
#define ESCOIN_MFMA(ACC, SET, A, B, P, Q)                                                                                    \
    ESCOIN_FENCE                                                                                                        \
    ACC[P][Q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, SET.p[P][A]), B##Q, ACC[P][Q], 0, 0, 0); \
    ESCOIN_FENCE
            // ROW: the tap's inputs; SET: its weights; CN: the set that the ones asked for now go to
#define ESCOIN_STEP(ROW, SET, CN, FURTHER, NOW, NEXT, NEXT_ROW)                                                         \
    __builtin_amdgcn_s_waitcnt(STAGE ? 0x4f74 : 0x0f74);                                                              \
    ESCOIN_MFMA(big, SET, 0, xh, 0, 0)                                                                                \
    xl0 = *(const h8*)(ROW + part);                                                                                   \
    ESCOIN_MFMA(big, SET, 0, xh, 0, 1)                                                                                \
    xl1 = *(const h8*)(ROW + part + 512);                                                                             \
    ESCOIN_MFMA(big, SET, 0, xh, 1, 0)                                                                                \
    weights(CN, 0, 0, FURTHER);                                                                                       \
    ESCOIN_MFMA(big, SET, 0, xh, 1, 1)                                                                                \
    weights(CN, 0, 1, FURTHER);                                                                                       \
    ESCOIN_MFMA(small, SET, 1, xh, 0, 0)                                                                              \
    weights(CN, 1, 0, FURTHER);                                                                                       \
    ESCOIN_MFMA(small, SET, 1, xh, 1, 0)                                                                              \
    xh0 = *(const h8*)(NEXT_ROW);                                                                                     \
    ESCOIN_MFMA(small, SET, 1, xh, 0, 1)                                                                              \
    weights(CN, 1, 1, FURTHER);                                                                                       \
    ESCOIN_MFMA(small, SET, 1, xh, 1, 1)                                                                              \
    xh1 = *(const h8*)((NEXT_ROW) + 512);                                                                             \
    __builtin_amdgcn_sched_barrier(0);                                                                                \
    ESCOIN_MFMA(small, SET, 0, xl, 0, 0)                                                                              \
    if (STAGE) fetch_four(NEXT, round + 1, First{});                                                                  \
    ESCOIN_MFMA(small, SET, 0, xl, 1, 0)                                                                              \
    if (STAGE) fetch_four(NEXT, round + 1, Second{});                                                                 \
    ESCOIN_MFMA(small, SET, 0, xl, 0, 1)                                                                              \
    ESCOIN_MFMA(small, SET, 0, xl, 1, 1)                                                                              \
    if (STAGE) {                                                                                                      \
        commit(NOW, other);                                                                                           \
        locate(NOW, ++task + 2);                                                                                      \
    }                                                                                                                 \
    ESCOIN_FENCE
            h8 xl0, xl1;
            const char* row1 = row + 16;
            const char* row2 = row + 32;
            if (STRIDE == 2) {
                row1 = base + tap_at(r, 1) * 16;
                row2 = row + 16;
            }
            const char* next_row = row + (++r == a.R ? sub_bytes - (a.R - 1) * a.pitch * 16 : a.pitch * 16);
            if (r == a.R) {
                r = 0;
                base += sub_bytes;
            }
            if (STRIDE == 2) next_row = base + tap_at(r, 0) * 16;
            ESCOIN_STEP(row, w0, w2, 0, ta, tc, row1)
            ask.next();
            ESCOIN_STEP(row1, w1, w0, 0, tb, ta, row2)
            ESCOIN_STEP(row2, w2, w1, kStepBytes, tc, tb, next_row)
            ask.at += 2 * kStepBytes;
            ask.left -= 2;
            row = next_row;
            i += 3;
#undef ESCOIN_STEP
#undef ESCOIN_MFMA
#undef ESCOIN_FENCE
        };
        const std::true_type with{};
        const std::false_type plain{};
        if (i < end) {
            xh0 = read(0, 0);
            xh1 = read(0, 1);
            if (a.S == 3 && s == 0 && (end - begin) % 3 == 0) {
                if (STRIDE == 1 && more && end - i >= in_threes)
                    while (task < in_threes) three(with);
                while (i < end) three(plain);
            }
            for (;;) {
                if (i == end) break;
                step(w0, w2);
                if (i == end) {
                    const Weights t = w0;
                    w0 = w1; w1 = w2; w2 = t;
                    break;
                }
                step(w1, w0);
                if (i == end) {
                    const Weights t = w0;
                    w0 = w2; w2 = w1; w1 = t;
                    break;
                }
                step(w2, w1);
            }
        }
        if (more) {
            if (STRIDE == 2) __syncthreads();  // the only window has been read
            // the tasks left over: two or three of them have been asked for
            if (task < my_tasks) commit(ta, other);
            if (task + 1 < my_tasks) commit(tb, other);
            if (three_ahead && 2 < my_tasks) commit(tc, other);
            for (task += three_ahead ? 3 : 2; task < my_tasks; ++task) {
                locate(ta, task);
                fetch(ta, round + 1);
                commit(ta, other);
            }
            locate(ta, 0);
            locate(tb, 1);
            locate(tc, 2);
            if (round + 2 < n_rounds) {
                fetch(ta, round + 2);
                fetch(tb, round + 2);
                if (three_ahead) fetch(tc, round + 2);
            }
        }
        // Long chains: the sums so far join the workgroup's in LDS (no registers are left for them), which makes two shares as exact as eight with
        // half their workgroups' beginnings (64x256x28x28 at 50 %: 224-240 -> 172-178 us; a flush costs some 600 clocks, all of them 4 %).
        // Half of a wave's channels at a time: the two waves that share them take one half each and change over, with a round's
        // barrier between, so neither waits for the other (a wave at a time: 178 us for 174).
        if (FLUSH && more) {
            const int turn = (round + 1) % a.flush;
            const bool first = round + 1 < a.flush;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                if (turn != ((p ^ kg) & 1)) continue;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    f4 s = first ? (f4)(0.0f) : total[(8 * p + i) * 64];
#pragma unroll
                    for (int b = 0; b < 4; ++b) s[b] += big[p][i >> 2][4 * (i & 3) + b];
                    total[(8 * p + i) * 64] = s;
                }
                big[p][0] = (f16v)(0.0f);
                big[p][1] = (f16v)(0.0f);
            }
        }
        __syncthreads();
    }
    if (lost) atomicAdd(&notes->lost, lost);

    // ---- the waves' sums over their channels meet in LDS (the window is dead): each finishes a share of the outputs
    constexpr int kShare = 64 / KW;
    auto part = [&](int i) ESCOIN_INLINE { return fmaf(0x1p-11f, small[i >> 5][i >> 4 & 1][i & 15], big[i >> 5][i >> 4 & 1][i & 15]); };
    f4* const meet = (f4*)win + (wm * PW + wp) * KW * (KW - 1) * (kShare / 4) * 64 + lane;
#pragma unroll
    for (int j = 0; j < KW; ++j) {
        if (j == kg) {
#pragma unroll
            for (int i = 0; i < kShare; ++i) v[i] = part(j * kShare + i);
        } else {
            f4* const o = meet + (j * (KW - 1) + (kg > j ? kg - 1 : kg)) * (kShare / 4) * 64;
#pragma unroll
            for (int i = 0; i < kShare / 4; ++i) {
                f4 s;
#pragma unroll
                for (int b = 0; b < 4; ++b) s[b] = part(j * kShare + 4 * i + b);
                o[i * 64] = s;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KW - 1; ++k) {
        const f4* const o = meet + (kg * (KW - 1) + k) * (kShare / 4) * 64;
#pragma unroll
        for (int i = 0; i < kShare / 4; ++i) {
            const f4 s = o[i * 64];
#pragma unroll
            for (int b = 0; b < 4; ++b) v[4 * i + b] += s[b];
        }
    }
    if (FLUSH) {
#pragma unroll
        for (int i = 0; i < kShare / 4; ++i) {
            const f4 s = total[(kg * (kShare / 4) + i) * 64];
#pragma unroll
            for (int b = 0; b < 4; ++b) v[4 * i + b] += s[b];
        }
    }

    // an input below 2^-13 is off by 2^-36 at most, a weight below 2^15: they matter to sums this small
    const float small_sum = 16.0f * (float)notes->lost;
    constexpr int kTiles = kShare > 16 ? kShare / 16 : 1, kEach = kShare / kTiles;
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
        const int tile = (kg * kShare + t * kEach) / 16;
        const bool inside = room.out_at()[wp * 64 + (tile & 1) * 32 + (lane & 31)] >= 0;
        const int m = mg * TM + wm * 64 + (tile >> 1) * 32 + 4 * (lane >> 5) + (kEach < 16 ? 2 * (kg * kShare % 16) : 0);
        bool bad = false;
#pragma unroll
        for (int i = 0; i < kEach; ++i)
            bad |= m + 8 * (i / 4) + i % 4 < a.M && !(fabsf(v[t * kEach + i]) <= FLT_MAX && fabsf(v[t * kEach + i]) >= small_sum);
        const uint64_t lanes = __ballot(bad && inside);
        if (__builtin_expect(lanes != 0, 0)) {
            if (lane == 0) atomicOr((unsigned long long*)&notes->again[wp], ((lanes | lanes >> 32) & 0xffffffffu) << (32 * (tile & 1)));
            uint64_t rows = 0;
            bool over = false;
#pragma unroll
            for (int i = 0; i < kEach; ++i) {
                const int k = m + 8 * (i / 4) + i % 4;
                const bool finite = fabsf(v[t * kEach + i]) <= FLT_MAX;
                rows |= k < a.M && !(finite && fabsf(v[t * kEach + i]) >= small_sum) ? 1ull << ((k - mg * TM) & 63) : 0ull;
                over |= k < a.M && !finite;
            }
            if (inside && rows != 0) atomicOr((unsigned long long*)&notes->rows[wm], rows);
            if (inside && over) notes->over = 1;
        }
    }
    __syncthreads();  // before the stores: nothing waits for those unless some outputs are computed again
    uint64_t any = 0;
#pragma unroll
    for (int run = 0; run < PW; ++run) any |= notes->again[run];
    *scale = ex;
    return any;
}

// Behind the window's table, in the dead window: a run of positions that read as zero.
template <int PW, class R>
__device__ inline void nowhere_past_the_table(const R& room, int lane, int wave) {
    if (wave < PW) room.tab()[room.WR + 64 * wave + lane] = kNowhere;
}

// The channels that are too short for pairs to be as exact as fp32 sums, from their nonzeros in fp32; the waves take them in turn.  A
// position's word for a tap stands in the window's table, so that a nonzero costs an LDS read, a load and a multiply-add; kFewBatch of
// them are in flight at once, a batch of a wave takes some 1200 clocks with all of them at it.  Bound by its instructions and the L1: with a test for
// the row's end and a lane number worked out for every nonzero a batch took 1600 (3x107x59x59, 388 channels, 170 batches: 77 -> 65 us, 41 without
// any), a batch fetched while the last one is summed made it no faster.  64x256x28x28, 80 %, rows of 55 to 2304 nonzeros: 184 us, with
// the short rows as pairs 148 and 1 to 2 % less exact than the tiled kernel, which takes 314.
template <int MW, int PW, int KW, int STRIDE>
__device__ inline void few_rows(const PairArgs& a, const Room<MW, PW> room, Rsrc in, int lane, int wave, int mg, int t0) {
    constexpr int kWaves = MW * PW * KW, TM = 64 * MW;
    const int EF = a.E * a.F, HW4 = a.H * a.W * 4, n_first = t0 / a.plane;
    const bool relu = a.flags & ESCOIN_F_RELU, has_bias = a.flags & ESCOIN_F_BIAS;
    const char* const tab = (const char*)(room.tab() + lane);
    int turn = 0;
    for (int m0 = mg * TM; m0 < min((mg + 1) * TM, a.M); m0 += 64) {
        int begin = 0, end = 0;
        if (m0 + lane < a.M) {
            begin = a.rowptr[m0 + lane];
            end = a.rowptr[m0 + lane + 1];
        }
        for (uint64_t list = __ballot(m0 + lane < a.M && end - begin < a.few); list != 0; list &= list - 1) {
            if (turn++ % kWaves != wave) continue;
            const int k = __ffsll((unsigned long long)list) - 1, m = m0 + k;
            const int last = __builtin_amdgcn_readlane(end, k);
            float v[PW][kFewChains] = {};
            for (int j = __builtin_amdgcn_readlane(begin, k); j < last; j += 64) {
                const int here = min(last - j, 64);
                const uint32_t* const p = (const uint32_t*)a.nz + 3 * (j + min(lane, here - 1));  // a nonzero a lane
                const uint32_t c = p[0], rs = p[1], value = p[2];
                const bool there = lane < here;  // past the end zeros meet
                const int r = rs & 0xffffu, s = rs >> 16;
                int tap = r * a.pitch + s;
                if (STRIDE == 2) tap = a.phase_at[2 * (r & 1) + (s & 1)] + (r >> 1) * a.pitch + (s >> 1);
                const uint32_t reach = 4u * (there ? tap : a.WR);
                const int channel = there ? (int)c * HW4 : 0, w = there ? (int)value : 0;
#pragma unroll
                for (int i = 0; i < 64; i += kFewBatch) {  // lane numbers are constants, which saves an instruction each
                    if (i >= here) break;
                    uint32_t src[kFewBatch][PW];
                    float x[kFewBatch][PW];
#pragma unroll
                    for (int b = 0; b < kFewBatch; ++b) {
                        const char* const t = tab + __builtin_amdgcn_readlane(reach, i + b);
#pragma unroll
                        for (int run = 0; run < PW; ++run) src[b][run] = *(const uint32_t*)(t + 256 * run);
                    }
#pragma unroll
                    for (int b = 0; b < kFewBatch; ++b)
#pragma unroll
                        for (int run = 0; run < PW; ++run)
                            x[b][run] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(in, src[b][run], __builtin_amdgcn_readlane(channel, i + b), 0));
                    __builtin_amdgcn_sched_barrier(0);  // all on their way before the first is waited for
#pragma unroll
                    for (int b = 0; b < kFewBatch; ++b)
#pragma unroll
                        for (int run = 0; run < PW; ++run)
                            v[run][b % kFewChains] = fmaf(__int_as_float(__builtin_amdgcn_readlane(w, i + b)), x[b][run], v[run][b % kFewChains]);
                }
            }
#pragma unroll
            for (int run = 0; run < PW; ++run) {
                const int at = room.out_at()[64 * run + lane];
                float y = (v[run][0] + v[run][1]) + (v[run][2] + v[run][3]);
                y += has_bias ? a.bias[m] : 0.0f;
                if (relu) y = y > 0.0f ? y : 0.0f;
                if (at >= 0) a.out[((size_t)n_first * a.M + m) * EF + at] = y;
            }
        }
    }
}

// MW, PW: waves over channels and positions, 64 each; KW: over the input channels, 16 each a round.
template <int MW, int PW, int KW, bool FLUSH, int STRIDE>
__global__ __launch_bounds__(64 * MW * PW * KW, 2) void sconv_pair_kernel(const PairArgs a) {
    constexpr int kWaves = MW * PW * KW, kThreads = 64 * kWaves, TP = 64 * PW, TM = 64 * MW;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int jobs = a.n_tiles * a.n_mgroups, jq = jobs >> 3, jr = jobs & 7;
    if (slot >= jq + (xcd < jr ? 1 : 0)) return;  // the whole workgroup, before any barrier
    const int job = xcd * jq + min(xcd, jr) + slot;
    const int tile = job / a.n_mgroups, mg = job - tile * a.n_mgroups;
    const int t0 = tile * TP;
    const int HW = a.H * a.W, CHW = a.C * HW, EF = a.E * a.F;
    const bool relu = a.flags & ESCOIN_F_RELU, has_bias = a.flags & ESCOIN_F_BIAS;

    const Room<MW, PW> room = {lds, a.WR};
    Notes<PW>* const notes = room.notes();
    const int row = min(mg * TM + tid, a.M - 1);
    int row_exp = 0;
    float row_bias = 0.0f;
    if (tid < TM) {
        row_exp = a.exps[row];
        if (has_bias) row_bias = a.bias[row];
    }
    const int n_first = t0 / a.plane, u_first = t0 - n_first * a.plane;
    const float one_over_plane = 1.0f / (float)a.plane, one_over_pitch = 1.0f / (float)a.pitch;
    for (int i = tid; i < a.WR; i += kThreads) {
        int rem, col;
        int u = u_first + i, odd_row = 0, odd_col = 0;
        if (STRIDE == 2) {
            odd_row = i >= a.phase_at[2] ? 1 : 0;
            odd_col = i >= (odd_row ? a.phase_at[3] : a.phase_at[1]) ? 1 : 0;
            u -= odd_row ? (odd_col ? a.phase_at[3] : a.phase_at[2]) : (odd_col ? a.phase_at[1] : 0);
        }
        const int n = divide(u, a.plane, one_over_plane, &rem), line = divide(rem, a.pitch, one_over_pitch, &col);
        const int y = STRIDE * line + odd_row - a.pad, x = STRIDE * col + odd_col - a.pad;
        const bool there = n_first + n < a.N;
        const bool inside = y >= 0 && x >= 0 && (STRIDE == 1 || (y < a.H && x < a.W));
        room.tab()[i] = there && inside ? (uint32_t)(n * CHW + y * a.W + x) * 4u : kNowhere;
        if (i < TP) room.out_at()[i] = there && line < a.E && col < a.F ? n * a.M * EF + line * a.F + col : -1;
    }
    if (tid < TM) {
        room.row_exp()[tid] = row_exp;
        room.row_bias()[tid] = row_bias;
    }
    if (tid < PW) notes->again[tid] = 0;
    if (tid == PW) notes->lost = 0;
    if (tid == PW + 1) notes->peak = 0;
    if (tid == PW + 2) notes->over = 0;
    if (tid >= PW + 3 && tid < PW + 5) notes->rows[tid - PW - 3] = 0;
    const size_t left = (size_t)(a.N - n_first) * CHW * 4;
    const Rsrc in = rsrc_of(a.in + (size_t)n_first * CHW, (uint32_t)min(left, (size_t)kNowhere));
    const Rsrc wr = rsrc_of(a.w, a.w_bytes);
    __syncthreads();

    constexpr int kShare = 64 / KW, kTiles = kShare > 16 ? kShare / 16 : 1, kEach = kShare / kTiles;
    const auto store = [&](const float (&v)[kShare], int ex) ESCOIN_INLINE {
        // A lane holds, per 32 positions, 16 output channels of one position: 8*(i/4) + 4*(lane/32) + i%4.
        const int wp = wave % PW, kg = wave / PW % KW, wm = wave / (PW * KW);
#pragma unroll
        for (int t = 0; t < kTiles; ++t) {
            const int sub = (kg * kShare + t * kEach) / 16, i0 = (kg * kShare) % 16;  // 32x32 tile of the wave; its first value
            const int at = room.out_at()[wp * 64 + (sub & 1) * 32 + (lane & 31)];
            const int m0 = wm * 64 + (sub >> 1) * 32 + 4 * (lane >> 5) + (kEach < 16 ? 2 * i0 : 0);
            if (at < 0) continue;
            float* __restrict__ o = a.out + ((size_t)n_first * a.M + mg * TM + m0) * EF + at;
            const int rows = a.M - mg * TM - m0;  // channels from this lane's first one on
#pragma unroll
            for (int i = 0; i < kEach; i += 4) {
                const i4 e = *(const i4*)(room.row_exp() + m0 + 2 * i);
                const f4 b = *(const f4*)(room.row_bias() + m0 + 2 * i);
                f4 y;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    y[k] = ldexpf(v[t * kEach + i + k], -ex - e[k]) + b[k];
                    if (relu) y[k] = y[k] > 0.0f ? y[k] : 0.0f;
                }
                if (2 * i + 4 <= rows) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) o[(size_t)(2 * i + k) * EF] = y[k];
                } else {
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if (2 * i + k < rows) o[(size_t)(2 * i + k) * EF] = y[k];
                }
            }
        }
    };
    enum { kDone, kNonzeros, kOnceMore } then = kDone;  // what some sums still need
    {
        float v[kShare];
        int ex;
        const uint64_t any = pass<MW, PW, KW, FLUSH, STRIDE, false>(a, room, in, wr, lane, wave, mg, v, &ex);
        // Said so that the usual way out is one piece of code (32x64x56x56: 33.9 -> 33.6 us); said for certain, the second pass is
        // compiled as one that never runs, with 150-200 registers spilled (inputs that need it: 0.42 -> 0.56 ms at 64x256x28x28).
        if (__builtin_expect_with_probability(any == 0, 1, 0.9)) {
            store(v, ex);
            if (__builtin_expect_with_probability(a.few == 0, 1, 0.7)) return;
        } else {
            int count = 0;
#pragma unroll
            for (int run = 0; run < PW; ++run) count += __popcll(notes->again[run]);
            then = __builtin_amdgcn_readfirstlane(notes->over != 0 || count > kFewBad ? 1 : 0) ? kOnceMore : kNonzeros;
            if (then == kNonzeros) store(v, ex);
        }
    }
    // What comes now is rare.  It reads the kernel's arguments, of which PairArgs is all, once more from where the launch put them, so that none has
    // to outlive the first pass: with them kept, 64 to 212 scalar registers were spilled, now 38 to 80, and the usual way through is 1-2 % faster
    // (32x64x56x56: 34.0 -> 33.5 us, 64x384x13x13 at 65 %: 107.2 -> 105.7, 64x256x28x28 at 50 %: 170.4 -> 169.2).  Some of what is rare takes 1-3 % longer
    // (a second pass at stride 2 everywhere: 132 -> 135 us; one sum from the nonzeros: 70.6 -> 72.9).
    int start = t0;
    auto from = (const __attribute__((address_space(4))) PairArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(start), "+s"(from));
    const PairArgs& b = *(const PairArgs*)from;
    const Room<MW, PW> room2 = {lds, b.WR};
    // (Said to be the same in all lanes: descriptors that might not be are read lane by lane.)
    const int n_first2 = __builtin_amdgcn_readfirstlane(start / b.plane), CHW2 = b.C * b.H * b.W;
    const uint32_t in_bytes = __builtin_amdgcn_readfirstlane((uint32_t)min((size_t)(b.N - n_first2) * CHW2 * 4, (size_t)kNowhere));
    const Rsrc in2 = rsrc_of(b.in + (size_t)n_first2 * CHW2, in_bytes), wr2 = rsrc_of(b.w, b.w_bytes);
    uint64_t any = then != kDone ? 1 : 0;
    // Perhaps an input was past the scale that the first ones asked for: once more with the scale of the largest.  Not where a few sums are
    // only too small for the bits that some input lost, as happens now and then behind a ReLU (one such sum in a launch of 32x128x56x56 at stride
    // 2: 38 -> 100 us with the second pass and all channels from their nonzeros).
    if (then == kOnceMore) {
        uint32_t most = 0;
        for (int i = tid; i < b.C * b.WR; i += kThreads) {
            const int c = i / b.WR;
            const uint32_t src = room2.tab()[i - c * b.WR];
            const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(in2, src == kNowhere ? src : src + (uint32_t)(c * b.H * b.W) * 4u, 0, 0) & 0x7fffffffu;
            most = max(most, x < 0x7f800000u ? +x : 0u);
        }
        __syncthreads();  // every wave has read the notes
        if (tid < PW) notes->again[tid] = 0;
        if (tid == PW) notes->lost = 0;
        if (tid >= PW + 3 && tid < PW + 5) notes->rows[tid - PW - 3] = 0;
        atomicMax(&notes->peak, most);
        __syncthreads();
        float v[kShare];
        int ex, lane2 = lane, wave2 = wave;
        asm volatile("" : "+v"(lane2));  // what the first pass made of it is not worth keeping for this one
        any = pass<MW, PW, KW, FLUSH, STRIDE, true>(b, room2, in2, wr2, lane2, wave2, mg, v, &ex);
        store(v, ex);
    }
    if (any != 0) {
        uint64_t lists[PW];
#pragma unroll
        for (int run = 0; run < PW; ++run) lists[run] = notes->again[run];
        __syncthreads();  // those stores before the ones of redo()
        redo(b, lists, start, mg * TM, TM, kWaves, wave, lane, notes->rows);
    }
    if (b.few != 0) {
        nowhere_past_the_table<PW>(room2, lane, wave);
        __syncthreads();  // and these
        few_rows<MW, PW, KW, STRIDE>(b, room2, in2, lane, wave, mg, start);
    }
}

template <int MW, int PW, int KW, bool FLUSH, int STRIDE>
int launch_shape(PairArgs& a, const Dims& d, hipStream_t stream) {
    const PairShape shape = {MW, PW, KW, a.few, a.flush};
    static_assert(sizeof(Notes<PW>) <= 64, "");
    a.n_mgroups = (d.M + 64 * MW - 1) / (64 * MW);
    a.n_tiles = (int)(((long long)d.N * a.plane + 64 * PW - 1) / (64 * PW));
    a.WR = pair_window(d, shape);
    a.groups = (a.WR + 63) / 64;
    for (int phase = 0; phase < 4; ++phase) a.phase_at[phase] = pair_phase_at(d, shape, phase);
    const int lds = pair_lds_bytes(d, shape);
    if (lds > kPairLdsBytes) return ESCOIN_ERANGE;
    a.total_at = lds - MW * PW * 64 * 256 - pair_head_bytes(shape) - 4 * a.WR;
    if (lds > 64 * 1024) {
        const int rc = allow_dynamic_lds((const void*)sconv_pair_kernel<MW, PW, KW, FLUSH, STRIDE>, lds);
        if (rc != ESCOIN_OK) return rc;
    }
    const unsigned blocks = (unsigned)(((long long)a.n_tiles * a.n_mgroups + 7) / 8 * 8);
    return launch(sconv_pair_kernel<MW, PW, KW, FLUSH, STRIDE>, dim3(blocks), dim3(64 * MW * PW * KW), (size_t)lds, stream, a);
}

template <int MW, int PW, int KW>
int start(PairArgs& a, const Dims& d, hipStream_t stream) {
    if (a.flush && (KW != 2 || d.stride == 2)) return ESCOIN_EINVAL;  // there is no such form
    if constexpr (KW < 8)
        if (d.stride == 2) return launch_shape<MW, PW, KW, false, 2>(a, d, stream);
    if (KW == 2 && a.flush) return launch_shape<MW, PW, KW, KW == 2, 1>(a, d, stream);
    return launch_shape<MW, PW, KW, false, 1>(a, d, stream);
}

}  // namespace

int launch_sconv_pair(const Dims& d, const PlanHeader& h, const PairShape& s, const char* d_plan, const float* d_in, float* d_out,
                      const float* d_bias, uint32_t flags, hipStream_t stream) {
    if (first_layer(d)) return launch_sconv_first(d, h, s.few, d_plan, d_in, d_out, d_bias, flags, stream);
    PairArgs a;
    const char* const section = d_plan + h.off_pair;
    a.in = d_in; a.out = d_out; a.bias = d_bias; a.flags = flags;
    a.w = (const b8*)section;
    a.w_bytes = (uint32_t)pair_weight_bytes(d);
    a.exps = (const int32_t*)(section + pair_weight_bytes(d));
    a.rowptr = (const int32_t*)(d_plan + h.off_nz);
    a.nz = (const MfmaNz*)(d_plan + h.off_nz + mfma_rowptr_bytes(d));
    a.N = d.N; a.C = d.C; a.H = d.H; a.W = d.W; a.M = d.M; a.E = d.E; a.F = d.F; a.R = d.R; a.S = d.S; a.pad = d.pad; a.stride = d.stride;
    a.pitch = pair_pitch(d);
    a.plane = (int)pair_plane(d);
    a.n_chunks = (int)mfma_chunks(d);
    a.few = s.few;
    a.flush = s.flush;
    const int layout = 100 * s.MW + 10 * s.PW + s.KW;
    if (layout == 114) return start<1, 1, 4>(a, d, stream);
    if (layout == 118 && d.stride == 1) return start<1, 1, 8>(a, d, stream);
    if (layout == 122) return start<1, 2, 2>(a, d, stream);
    if (layout == 212) return start<2, 1, 2>(a, d, stream);
    return ESCOIN_EINVAL;
}

}  // namespace escoin
