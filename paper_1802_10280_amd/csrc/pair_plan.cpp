// Host side of the fp16-pair form: which layers have one, and its section of the plan.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "pair.h"

namespace escoin {

// The layouts there are.  On a large layer (64x256x28x28, 256 3x3 filters) they take, in this order, 179, 245, 167 and
// 162 us; on small ones the order turns round: 512 channels of 7x7, batch 32: 35, 33, 62, 57.
static const PairShape kShapes[] = {{1, 1, 4}, {1, 1, 8}, {1, 2, 2}, {2, 1, 2}};

// Fewer workgroups leave most compute units idle, where the tiled kernel has smaller ones.
constexpr double kLeastJobs = 64;

// Microseconds that a batch of N images takes in one of the layouts.  A workgroup takes 12000 clocks to begin and to
// end (17000 in a launch of several rounds of them) and, with another one beside it or not, 900 a step (1180 with eight
// waves) and 250 a staging task, where filters are three wide; with others 1150 a step and, for
// a round, staged without overlap, 2700 and 750 a task.  The last workgroups to run count for more than their share.  2 GHz,
// as measured over launches of this length.  That is 157, 33, 31, 26 and 96 us where 162, 37, 33, 30 and 100 were measured (28x28
// with 256 channels, 56x56 with 64, 7x7 with 512, 14x14 with 256, 13x13 with 384) and 18, 10 and 12 where 19, 11 and 12
// were (13 of 15x15 with 240, one of 41x44 with 24, 5 of 7x7 with 69).
//
// At stride 2 the next round is staged when the last one is over.  A workgroup that has a compute unit to itself takes 16800 clocks around its
// steps and 600 a step, beside another one 26000 and 900; 620 a staging task, and 2300 a round where filters are not three wide.  That is
// 25, 24, 26, 43, 33, 14 and 104 us where 26, 26, 25, 41, 30, 13 and 100 were measured (32 images of 56x56 with 64 channels, 28x28 with 128 in both layouts,
// 14x14 with 256 in both; 13 of 63x63 with 30; 64 of 31x31 with 128, 5x5; tiled: 40, 43, 43, 53, 53, 18, 195).  Where a workgroup leaves no room for another one a last
// round takes as long as a whole one, however few they are (266 to 342 workgroups with filters five wide: 2.0 to 2.1 times as long as 256).
//
// `few`: batches of nonzeros of all short rows.  A batch takes a wave 1200 clocks for 64 positions, with all of them at it; counted as 1900, since
// a whole row falls to one wave.  105 random layers of uneven rows that take the pairs by this need 0.39 to 0.96 of the tiled kernel's time, one
// 1.09 (26 of 25x25, 34 -> 51 channels, 5x5: 22.4 us and 31.3, but 34.0 for inputs that send one workgroup through its second pass).  At stride 2 a launch of one
// round is as long as the workgroup that has a short row, of four batches or so (12 of 18x26x26, 371 3x3 filters: 13 us by the mean, 16 measured).
static double pair_time(const Dims& d, double N, const PairShape& s, double few = 0) {
    const int waves = s.MW * s.PW * s.KW, lds = pair_lds_bytes(d, s), RS = d.R * d.S;
    if (lds > kPairLdsBytes || (d.stride == 2 && waves > 4)) return INFINITY;
    const double jobs = ceil(N * (double)pair_plane(d) / (64 * s.PW)) * ceil(d.M / (64.0 * s.MW));
    if (jobs < kLeastJobs) return INFINITY;
    const double slots = waves == 4 && 2 * lds <= kPairLdsBytes ? 512 : 256;
    const int chunks = (int)mfma_chunks(d), rounds = (chunks + s.KW - 1) / s.KW;
    const double steps = ceil((double)chunks * RS / s.KW), tasks = ceil(2.0 * s.KW * ((pair_window(d, s) + 63) / 64) / waves);
    double job = jobs > slots ? 17000 : 12000;
    if (d.stride == 2) {
        const bool shared = jobs > 256 && slots == 512;
        job = (shared ? 26000 : 16800) + steps * (shared ? 900 : 600) + (rounds - 1) * (tasks * 620 + (d.S == 3 ? 0 : 2300));
    } else if (d.S == 3) job += steps * (waves == 4 ? 900 : 1180) + (rounds - 1) * tasks * 250;
    else job += steps * 1150 + (rounds - 1) * (2700 + tasks * 750);
    if (s.flush) job += rounds / s.flush * 700;
    const double batches = few / ceil(d.M / (64.0 * s.MW)) / waves * 1900;
    job += s.PW * (d.stride == 2 && few > 0 && jobs <= slots ? std::max(batches, 4 * 1200.0) : batches);
    const double full = floor(jobs / slots), rest = jobs / slots - full;
    return 2.0 + std::max(1.0, full + (rest > 0 ? (d.stride == 2 && slots == 256 ? 1.0 : 0.5 + 0.5 * rest) : 0.0)) * job / 2000.0;
}

// The tiled kernel's, from its tiling: rounds of workgroups over 8 x 32 compute units; a workgroup's 4 us and half a us a chunk, and the
// LDS reads of its records, 4.6 clocks of 2.1 GHz for each position run and half of that for the record itself.  That is 48, 48, 56,
// 58, 188 and 107 us where 48, 47, 55, 59, 177 and 111 were measured (56x56 with 64 channels, 28x28 with 128, 14x14 with 256, 7x7 with 512,
// 28x28 with 256 at 90 and 95 %), 11 and 12 where 11 and 15 were (16 channels, 5x5; 192 channels, 1x1).  At stride 2 it takes a fifth more: 38, 41, 47, 70, 213, 17 where
// 40, 43, 53, 58, 195 and 18 were (the layers above).  Not with few channels, whose chunks are few: with 2 us for the launch, 52, 194, 125, 28, 136 and 58 where 50, 197, 122, 28,
// 130 and 57 were (5 and 32 images of 3x224x224, 64 7x7 filters; 12 of 2x236x236, 63 11x11; 20 of 4x61x61, 128 6x6; 40 of 3x182x60, 53 11x11; 64 of 1x64x200, 100
// 9x9 of stride 4; all at 30 %, but the last at 10).
static double tiled_time(const Dims& d, double N, const PlanHeader& h) {
    const double jobs = (double)h.n_tiles * ceil(N / h.NB) * h.n_mgroups * h.CS;
    const double job = 4.0 + 0.5 * h.n_chunks / h.CS + (double)h.n_records / h.n_mgroups / h.CS * h.WQ * (h.Q + 0.5) * 4.6 / 2100.0;
    return ceil(ceil(jobs / 8) / 32) * job * (d.stride == 2 && !first_layer(d) ? 1.2 : 1.0);
}

// How much faster it has to look, as the estimates are off by a tenth now and then.
constexpr double kMargin = 0.9;

// The shapes the kernel takes.
static bool pair_takes(const Dims& d) {
    if (d.stride > 2 || (d.stride == 1 && (d.R <= d.pad || d.S <= d.pad)) || d.C < 16 || d.M < 32) return false;
    if (pair_reach(d) > kPairReach || pair_weight_bytes(d) > (64ull << 20)) return false;
    // positions, and the offsets inside the images that a workgroup's window may touch, in 32 bits; and those of the channels that a round
    // of four chunks asks for past the last one, before they are held to it (where an image of two million positions at stride 2 has four times as
    // many inputs; at stride 1 even eight chunks stay below)
    const long long plane = pair_plane(d), images = (128 + kPairReach) / plane + 2;
    if ((d.C + 63ll) / 64 * 64 * d.H * d.W * 4 >= (1ll << 31)) return false;
    return plane < (1 << 21) && images * d.C * d.H * d.W * 4 < (1ll << 31) && images * d.M * d.E * d.F < (1ll << 31);
}

// Relative errors against 64 bits, squared, times 1e14 (2-norm; n nonzeros a row, activations half zeros).  Two fp16
// numbers hold 22 to 23 bits: with the product left out that makes 0.9e-7 whatever n is; the sums add to it, the less the more
// waves share them.  The tiled kernel's chains of fp32 roundings are n / WS long, the kernel of three bf16 parts
// rounds once per 16 channels.  Measured and (in brackets) by these, in 1e-7: pairs in two shares, n = 115: 1.12 (1.15), 460: 1.75
// (1.68); in four, 60: 0.97 (0.96), 460: 1.37 (1.32); in eight, 60: 0.99 (0.99), 920: 1.39 (1.37), 1210: 1.47 (1.48).  Tiled,
// 60: 0.99 (0.96), 115: 1.36 (1.33), 460: 2.64 (2.66).  bf16, 691: 1.16 (1.16), 1210: 1.54 (1.54).
// Over 60 random layers that take the pairs (1 to 64 images, 7 to 64 wide, 16 to 512 channels, 50 to 90 %, even and uneven rows, half of the
// inputs zeros) they err 0.25 to 0.86 times as much as the kernel they stand in for.
// Chains round once for each input that is not a zero, so all of this is for activations as a ReLU leaves them.  With sparser ones
// the pairs' share stays (0.8e-7 at 3 %) while the chains' falls: they are even at 43 % where the pairs stand in for three bf16 parts and at 7
// to 30 % where they do for the tiled kernel, and at 3 % a layer of 115 is at 0.84 and 0.42.  The kernel sees the inputs too late, so who has
// such inputs, and needs those bits, fixes a tuning.
// Two shares whose sums are flushed as often as flush_rounds() says are taken for eight, whose chains are as long: measured 1.33 and 1.38 (256
// channels, 3x3, 50 %), 1.39 and 1.44 (384, 65 %).
static double pair_base(const PairShape& s) { return s.KW == 8 || s.flush ? 0.92 : 0.81; }
static double pair_slope(const PairShape& s) { return s.KW == 8 || s.flush ? 0.00105 : s.KW == 4 ? 0.0020 : 0.0044; }
static double tiled_slope(int WS) { return 0.0154 / WS; }
constexpr double kTiledRowSlope = 0.0163, kMfmaSlope = 0.00195;  // the first: a row of 36 to 90 nonzeros, WS = 1
static double pair_error(double n, const PairShape& s) { return pair_base(s) + pair_slope(s) * n; }

// Rounds between a wave's flushes: such that its chains are as long as with eight shares, and as exact.  0 where the wave and its partner would not
// both have had a turn by then, for launches that do not fill every compute unit twice, where eight shares are as fast (32 images of
// 13x13, 512 channels, 384 filters at 50 %: 93.4 us both ways), and at stride 2, whose kernels flush nothing: where two shares are not exact
// enough there, as beside the split rows of a plan made for few images, four are.
static int flush_rounds(const Dims& d, const PairShape& s) {
    if (d.stride != 1 || s.KW != 2 || ceil(d.N * (double)pair_plane(d) / (64 * s.PW)) * ceil(d.M / (64.0 * s.MW)) < 512) return 0;
    const int flush = (int)mfma_chunks(d) / 8;
    return flush >= 2 ? flush : 0;
}

// A row of fewer nonzeros is less exact as pairs than in a kernel of that slope.
static int least_row(const PairShape& s, double slope) {
    const double gain = slope - pair_slope(s);
    return (int)std::min(ceil(pair_base(s) / std::max(gain, 1e-9)), 1e9);
}

// Layers of few channels: the shapes their kernel takes, its time and its error (the pairs' own, and a rounding for each 8 products of two chains;
// inputs as of an image, none of them zero, make the chains of the tiled kernel twice as long as those this is weighed against).  Over 200 random layers
// whose inputs are half zeros the error was 0.7 to 1.2 times this, the tiled kernel's 0.9 to 1.15 times its own, so some room is left between them.
static bool first_takes(const Dims& d) {
    return d.stride % 2 == 0 && d.M >= 32 && (long long)d.C * d.H * d.W * 4 < (1ll << 31) && (long long)d.E * d.F < (1ll << 30) && first_columns(d) < (1 << 12) && first_in_rows(d) < (1 << 12) &&
           first_loads(d) <= kFirstLoads && first_steps(d) <= kFirstSteps;
}
static double first_error(const Dims& d) { return 0.5 + 0.0308 * (first_steps(d) + 2); }
// A row of fewer nonzeros is less exact as pairs (measured where half of the inputs are zeros: 0.93e-7 and 0.97e-7 at 59 a row, 0.92 and 0.90 at 50).
static int first_line(const Dims& d) { return (int)ceil(first_error(d) / kTiledRowSlope); }
// Microseconds; a workgroup beside another one takes three fifths as long again, so the first of a further round of 256 cost more than their share.  17, 85,
// 49, 22, 17, 43, 26 and 57 where 18, 79, 51, 22, 16, 41, 24 and 53 were measured (the layers named at tiled_time(), the third with 4 images too; 16 of 6x120x120, 235
// 5x5); without short rows 320 random layers took at most 1.08 times as long as this.
// `few`: short rows.  One of up to 57 nonzeros keeps its wave for 12 us after all else, in two workgroups of a compute unit at once; many are bound by their
// gathers, 2 us a row and workgroup of a compute unit, 3 at stride 4.  1, 8 and 32 such rows of 64 take 12, 16 and 64 us more where 12, 19 and 63 were measured
// (5x3x224x224), 37, 98 and 392 where 40, 79 and 341 were (32 of them), 21, 55 and 220 where 22, 50 and 204 were (12x2x236x236, of 76 nonzeros), 11, 45 and
// 179 where 14, 45 and 185 were (stride 4).  Counted as 15.5, 3 and 4.5, as short rows do not spread evenly over workgroups, nor those over the XCDs: of
// 90 random layers with some, taken by this, one was slower than on the tiled kernel, by 3 %.
static double first_time(const Dims& d, double N, int few) {
    const double jobs = N * ceil((double)d.E * d.F / kFirstPositions) * ceil(d.M / 64.0), row = (first_line(d) - 1) / 57.0;
    const double most = few * std::min(64.0 / d.M, 1.0);  // of a workgroup's channels
    const double alone = 15.5 * ceil(most / 8) * std::max(1.0, jobs / 512), together = 0.75 * (2 + d.stride) * most * std::max(1.0, jobs / 256);
    const double full = floor(jobs / 256), rest = jobs / 256 - full;
    return 3.0 + std::max(1.15, full + (rest > 0 ? 0.6 + 0.4 * rest : 0.0)) * (7.5 + 0.4 * first_steps(d)) + row * std::max(alone, together);
}

// Whether a plan with this tiled form carries the section: a layer that some batch is faster with, and no less exact.
bool pair_planned(const Dims& d, long long nnz, const PlanHeader& h) {
    if (first_layer(d)) return first_takes(d) && first_error(d) < 0.92 * tiled_slope(h.WS) * (double)nnz / d.M;
    const double n = (double)nnz / d.M;
    if (!pair_takes(d)) return false;
    for (const PairShape& s : kShapes)
        for (double positions = 8192; pair_error(n, s) < 0.95 * tiled_slope(h.WS) * n && positions <= 8192 * 64; positions *= 4) {
            const double N = ceil(positions / (double)pair_plane(d));
            if (pair_time(d, N, s) < kMargin * tiled_time(d, N, h)) return true;
        }
    return false;
}

// Notes of the rows what pair_taken() asks.
void pair_note_rows(const Dims& d, const int32_t* rp, PlanHeader* h) {
    h->pair_least = INT32_MAX;
    for (int m = 0; m < d.M; ++m) h->pair_least = std::min(h->pair_least, rp[m + 1] - rp[m]);
    if (first_layer(d)) {
        h->pair_few2 = 0;
        for (int m = 0; m < d.M; ++m) h->pair_few2 += rp[m + 1] - rp[m] < first_line(d) ? 1 : 0;
        return;
    }
    for (const PairShape& s : kShapes) {
        const int least = least_row(s, kTiledRowSlope / h->WS);
        long long batches = 0;
        for (int m = 0; m < d.M; ++m)
            if (rp[m + 1] - rp[m] < least) batches += (rp[m + 1] - rp[m] + kFewBatch - 1) / kFewBatch;
        (s.KW == 2 ? h->pair_few2 : s.KW == 4 ? h->pair_few4 : h->pair_few8) = (int32_t)batches;
    }
}

// Whether a forward call on this batch takes the section of a plan made for this layer, and in which layout: one that is
// faster and no less exact than the kernel the call would take else, row by row.  Rows too short for the pairs are computed from their
// nonzeros in kFewChains chains, so where the tiled kernel has no more than those.  (Which kernel that is goes with the batch, and
// so does whether the pairs are exact enough: the results of a layer may change in their last bits from batch to batch, but
// no call's are less exact than without the pairs.)
bool pair_taken(const Dims& d, const PlanHeader& h, PairShape* shape) {
    if (h.pair != 1 || h.pair_least <= 0 || !pair_planned(d, h.pair_nnz, h)) return false;
    const long long total = (long long)d.N * pair_plane(d);
    if (total > (1ll << 30) || total / 64 * (long long)mfma_row_blocks(d) > (1ll << 30)) return false;
    if (first_layer(d)) {
        const double jobs = (double)d.N * ceil((double)d.E * d.F / kFirstPositions) * ceil(d.M / 64.0);
        *shape = {1, kFirstPositions / 64, 1, h.pair_least < first_line(d) ? first_line(d) : 0};
        if (h.WS > 1 && h.pair_least < first_line(d) * h.WS) return false;  // the tiled kernel's chains are shorter than those of short rows here
        return grid_fits(jobs, 2 * kFirstPositions) && first_time(d, d.N, h.pair_few2) < 2.0 + tiled_time(d, d.N, h);
    }
    const bool bf16 = mfma_taken(d, h);
    const double n = (double)h.pair_nnz / d.M, slope = bf16 ? kMfmaSlope : tiled_slope(h.WS);
    double best = kMargin * (bf16 ? mfma_time(d, d.N) : tiled_time(d, d.N, h));
    bool taken = false;
    for (PairShape s : kShapes) {
        const double most = (bf16 ? 1.0 : 0.95) * slope * n;
        if (pair_error(n, s) > most) s.flush = flush_rounds(d, s);
        if (pair_error(n, s) > most) continue;
        if (!grid_fits(ceil(total / (64.0 * s.PW)) * ceil(d.M / (64.0 * s.MW)), 64 * s.MW * s.PW * s.KW)) continue;
        const int least = least_row(s, bf16 ? kMfmaSlope : kTiledRowSlope / h.WS);
        const bool few = h.pair_least < least;
        if (few && (bf16 || h.WS > kFewChains || s.flush)) continue;
        // (With filters three wide flushed two shares are some 6 % slower than pair_time() has it, and eight up to 8 % faster: 37 of 377x29x29, 171 filters
        // took 163 and 157 us.)
        const double t = (s.flush && d.S == 3 ? 1.1 : 1.0) * pair_time(d, d.N, s, !few ? 0 : s.KW == 2 ? h.pair_few2 : s.KW == 4 ? h.pair_few4 : h.pair_few8);
        if (t < best) {
            best = t;
            *shape = s;
            shape->few = few ? least : 0;
            taken = true;
        }
    }
    return taken;
}

// x, below 2^15 in size, to the nearest fp16 number (ties to even); *back is its value
static uint16_t to_half(float x, float* back) {
    uint32_t u, sign;
    memcpy(&u, &x, 4);
    sign = u >> 16 & 0x8000u;
    u &= 0x7fffffffu;
    uint32_t h;
    float v;
    if (u < 0x38800000u) {  // below 2^-14: multiples of 2^-24, as the last bits of a sum with 1/2
        memcpy(&v, &u, 4);
        v += 0.5f;
        memcpy(&h, &v, 4);
        h -= 0x3f000000u;
        v -= 0.5f;
    } else {
        u += 0xfffu + (u >> 13 & 1u);
        u &= 0xffffe000u;
        h = (u >> 13) - (112u << 10);
        memcpy(&v, &u, 4);
    }
    *back = sign ? -v : v;
    return (uint16_t)(h | sign);
}

// Writes the weights and the rows' exponents into `out` (zeroed).  False where it cannot stand for the CSR: a value
// that is not finite, a row whose values span more than 27 binades (each row is scaled so that its largest lies below
// 2^15; the parts of one below 2^-13 would lose bits), or a row of fewer than 32 nonzeros, which fp32 rounds less often
// than this form errs.
bool pair_write(const Dims& d, const int32_t* rp, const MfmaNz* nz, char* out) {
    const size_t RS = (size_t)d.R * d.S, chunks = mfma_chunks(d);
    uint16_t* w = (uint16_t*)out;
    int32_t* exps = (int32_t*)(out + pair_weight_bytes(d));
    for (int m = 0; m < d.M; ++m) {
        if (rp[m + 1] - rp[m] < 32) return false;
        float most = 0.0f, least = INFINITY;
        for (int j = rp[m]; j < rp[m + 1]; ++j) {
            const float v = fabsf(nz[j].val);
            if (!(v < INFINITY)) return false;
            most = std::max(most, v);
            least = std::min(least, v);
        }
        exps[m] = 14 - ilogbf(most);
        if (ldexpf(least, exps[m]) < 0x1p-13f) return false;
        // in two factors: either may be past the largest float, or below the least, but not both
        const float up = ldexpf(1.0f, exps[m] / 2), up2 = ldexpf(1.0f, exps[m] - exps[m] / 2);
        for (int j = rp[m]; j < rp[m + 1]; ++j) {
            const float v = nz[j].val * up * up2;
            float high, rest;
            uint16_t part[2];
            part[0] = to_half(v, &high);
            part[1] = to_half((v - high) * 2048.0f, &rest);
            const int c = nz[j].c;
            size_t step = ((size_t)(m / 32) * chunks + c / 16) * RS + (size_t)nz[j].r * d.S + nz[j].s;
            size_t lane = m % 32 + 32 * (size_t)(c % 16 / 8), place = c % 8;
            if (first_layer(d)) {
                const size_t group = ((size_t)c * d.R + nz[j].r) * first_width(d) + nz[j].s / 8;
                step = (size_t)(m / 32) * first_steps(d) + group / 2;
                lane = m % 32 + 32 * (group % 2);
                place = nz[j].s % 8;
            }
            for (int k = 0; k < 2; ++k) w[((step * 2 + k) * 64 + lane) * 8 + place] = part[k];
        }
    }
    return true;
}

}  // namespace escoin
