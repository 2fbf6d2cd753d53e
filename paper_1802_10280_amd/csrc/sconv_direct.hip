// sconv, general form: Algorithm 2 on the stretched CSR and the padded input array, with the
// data-to-thread mapping of Section 3.2 (consecutive lanes own consecutive output positions,
// numbered through the images of the batch).  It accepts any filter size, stride and CSR entry
// order.  A wave owns one output channel: its CSR row is wave-uniform, so the (offset, value)
// pairs travel through the scalar data path instead of being staged in LDS; the input window is
// read through the vector L1/L2, which plays the part of the read-only cache of Section 3.3.
//
// What bounds it: with one nonzero at a time, the latency of its loads (about 380 clocks a nonzero in a small launch); with
// many in flight, the L1, which takes a wave's 64 words in 4 clocks at best.  Hence kAhead nonzeros' loads in flight, the next
// ones' (offset, value) pairs fetched meanwhile, and positions numbered so that four neighbouring lanes read four
// neighbouring words (see `pitch` at the launch).  Measured, one nonzero at a time -> this, in us: 128 -> 128 channels of 28x28,
// batch 32, 80 % sparse: 145 -> 100 (5.2 clocks a load and compute unit); 384 -> 384 of 13x13, batch 128: 2130 -> 1019;
// 271 -> 70 of 21x21, stride 2, one image: 200 -> 30.  Sums are formed in the CSR's order, as before: the same bits.
#include <algorithm>

#include "common.h"

namespace {

constexpr int kTail = 4;  // nonzeros at a time at the end of a row; the loads past it repeat the last one's

// A wave owns one output channel and 64 * kPix positions of a group of images, a workgroup kRows neighbouring channels.
// The positions of the group's images are numbered through (image, h, w), `pitch` to a row of the map, so that small maps
// fill the lanes as well as large ones.  Offsets inside a group fit 32 bits (the launch sizes the
// groups for that).
template <int kPix, int kAhead, int kRows>
__global__ __launch_bounds__(kRows * 64) void sconv_direct_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ value, const float* __restrict__ padded, float* __restrict__ out,
    const float* __restrict__ bias, uint32_t flags, int N, int M, int E, int F, int Wp, int pitch, int stride,
    int img_elems /* C*Hp*Wp */, int group_images, int n_groups, int bx, int deal) {
    // Workgroup -> (image group, output channel, block of positions), all channels of a group
    // before the next group.  Consecutive workgroup ids land on different XCDs (id mod 8), each
    // with an L2 of its own.  Small images: the XCDs share every group (plain order).  Large
    // images (`deal`): the groups are dealt to the XCDs in turn and an XCD walks its own groups
    // one after the other, so that the few groups it has in flight stay in its L2.
    const uint32_t per_group = (uint32_t)bx * (uint32_t)((M + kRows - 1) / kRows);
    uint32_t group, rest;
    if (deal) {
        const uint32_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        group = (slot / per_group) * 8 + xcd;
        rest = slot % per_group;
    } else {
        group = blockIdx.x / per_group;
        rest = blockIdx.x % per_group;
    }
    if (group >= (uint32_t)n_groups) return;
    const int m = (int)(rest / (uint32_t)bx) * kRows + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (m >= M) return;
    const uint32_t xblk = rest % (uint32_t)bx;
    const int EF = E * F, span = (E - 1) * pitch + F;
    const int j0 = rowptr[m], j1 = rowptr[m + 1];
    const float b = (flags & ESCOIN_F_BIAS) ? bias[m] : 0.0f;
    const int n_first = (int)group * group_images;
    const int n_here = min(group_images, N - n_first);
    const uint32_t positions = (uint32_t)n_here * (uint32_t)span;
    const float* __restrict__ grp = padded + (size_t)n_first * img_elems;
    if (xblk * (64 * kPix) >= positions) return;
    uint32_t p[kPix], base[kPix];
    float acc[kPix];
#pragma unroll
    for (int k = 0; k < kPix; ++k) {
        p[k] = (xblk * kPix + k) * 64 + (threadIdx.x & 63);
        const uint32_t pc = p[k] < positions ? p[k] : 0;  // clamp: out-of-range lanes read a valid pixel
        const uint32_t n = pc / (uint32_t)span, pp = pc - n * (uint32_t)span;
        const uint32_t h = pp / (uint32_t)pitch, w = pp - h * (uint32_t)pitch;
        base[k] = n * (uint32_t)img_elems + h * (uint32_t)(stride * Wp) + w * (uint32_t)stride;  // f(0, h, w) of image n
        acc[k] = b;
    }
    int j = j0;
    if (j + kAhead <= j1) {
        uint32_t off[kAhead];
        float val[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) off[u] = (uint32_t)colidx[j + u], val[u] = value[j + u];
        for (;;) {
            float x[kAhead][kPix], w[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int k = 0; k < kPix; ++k) x[u][k] = (grp + off[u])[base[k]];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) w[u] = val[u];
            j += kAhead;
            const bool more = j + kAhead <= j1;
            if (more) {
#pragma unroll
                for (int u = 0; u < kAhead; ++u) off[u] = (uint32_t)colidx[j + u], val[u] = value[j + u];
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int k = 0; k < kPix; ++k) acc[k] = fmaf(w[u], x[u][k], acc[k]);
            if (!more) break;
        }
    }
    for (; j < j1; j += kTail) {
        float x[kTail][kPix], w[kTail];
#pragma unroll
        for (int u = 0; u < kTail; ++u) {
            const int at = min(j + u, j1 - 1);
            const uint32_t off = (uint32_t)colidx[at];
            w[u] = value[at];
#pragma unroll
            for (int k = 0; k < kPix; ++k) x[u][k] = (grp + off)[base[k]];
        }
#pragma unroll
        for (int u = 0; u < kTail; ++u)
            if (j + u < j1) {
#pragma unroll
                for (int k = 0; k < kPix; ++k) acc[k] = fmaf(w[u], x[u][k], acc[k]);
            }
    }
#pragma unroll
    for (int k = 0; k < kPix; ++k) {
        float v = acc[k];
        if (flags & ESCOIN_F_RELU) v = v > 0.0f ? v : 0.0f;
        const uint32_t n = p[k] / (uint32_t)span, pp = p[k] - n * (uint32_t)span;
        const uint32_t h = pp / (uint32_t)pitch, w = pp - h * (uint32_t)pitch;
        if (p[k] < positions && w < (uint32_t)F) out[((size_t)(n_first + n) * M + m) * EF + h * (uint32_t)F + w] = v;
    }
}

}  // namespace

namespace escoin {

int launch_sconv_direct(const Dims& d, const int32_t* d_rowptr, const int32_t* d_colidx,
                        const float* d_value, const float* d_padded, float* d_out,
                        const float* d_bias, uint32_t flags, hipStream_t stream) {
    // Four positions a lane and eight nonzeros ahead, where the launch has waves to spare or the rows are so short that a
    // wave's setup shows; else one position, sixteen ahead and a workgroup of one wave, for more of them.  `waves`: of the
    // second kind, per SIMD.  Measured (first, second, us): 28x28, 128 -> 128, batch 32 (49 waves, dense rows of 1152):
    // 100, 120; 16x16, 16 -> 362, batch 16, 5x5 (22, 400): 10.9, 14.6; 10x59, 32 -> 363, batch 4 (13, 288): 29.7, 25.6;
    // 12x12, 296 -> 195, batch 18 (7.7, 2664): 75, 57; 19x19, 383 -> 35, one image (0.2, 3447): 80, 19.
    const double waves = (double)d.N * d.E * d.F * d.M / (64 * 1024);
    const bool four = waves >= 25 || 20 * waves >= (double)d.C * d.R * d.S;
    const int rows = four ? 4 : 1;
    // An L1 read takes four lanes of neighbouring words in one go.  Numbered through the outputs, positions keep to that only
    // if a row of the map is a multiple of four; else, for stride 1, through the padded rows, which leaves out the
    // last Wp - F of each row's lanes.  Measured (through the outputs, through the padded rows, us): 13x13, 384 -> 384, batch 128:
    // 2084, 1019; 19x19, 177 -> 268, batch 37: 956, 522; 28x28, 128 -> 128, batch 32: 100, 109; 16x16, 96 -> 336, batch 24: 86, 101; and
    // where the padding is over half of the map, 7x7 with 5x5, 440 -> 81, batch 6: 131, 141.
    const bool through_padded = d.stride == 1 && d.F % 4 && 2 * (long long)d.Wp < 3 * (long long)d.F;
    const long long pitch = through_padded ? d.Wp : d.F, EF = (long long)(d.E - 1) * pitch + d.F;
    const long long img_elems = (long long)d.C * d.Hp * d.Wp;
    // images per group: offsets inside a group (below group * img_elems, plus a nonzero's own
    // offset below img_elems) and position numbers stay under 2^32
    long long limit = std::max<long long>(1, std::min<long long>(d.N, ((1ll << 31) / img_elems)));
    limit = std::max<long long>(1, std::min<long long>(limit, (1ll << 30) / EF));
    // A group's padded input should stay in an L2 (4 MB per XCD) while all M output channels
    // walk over it, and its positions should fill the lanes of whole waves.  Where the images in flight are far more than
    // an L2 holds, and come near enough to a multiple of 8, they are dealt to the XCDs; a few XCDs with an image
    // more than the others cost more than the L2 gives.  Measured (dealt, plain, us): 64 images of 56x56, 256 -> 32: 362, 541;
    // 32 of 28x28, 128 -> 128 (8.3 MB in flight): 98, 101; 24 of 27x27, 100 -> 142 (7.1 MB): 167, 156; 37 of 19x19, 177 -> 268: 1134, 958;
    // 3 of 45x45, 88 -> 501: 350, 140.
    // Among the group sizes that split the batch evenly and hold at most 6 MB of input: the best lane fill (x XCD balance), ties
    // to the smaller.
    const long long per_block = four ? 256 : 64;
    const long long image_waves = (EF + per_block - 1) / per_block * ((d.M + rows - 1) / rows) * rows;
    const long long flying = std::min<long long>(d.N, 8192 / image_waves + 2);  // 32 waves a compute unit
    const bool deal = flying * img_elems * 4 > (15ll << 19) && 16 * (long long)d.N >= 15 * (((long long)d.N + 7) / 8 * 8);
    const long long most = std::max<long long>(1, std::min<long long>(limit, (6ll << 20) / (img_elems * 4)));
    long long group = 1;
    double best = 0.0;
    for (long long g = 1; g <= most; ++g) {
        const long long n_g = (d.N + g - 1) / g, even = (d.N + n_g - 1) / n_g;
        if (even != g) continue;
        const double fill = (double)(g * EF) / (double)(((g * EF + per_block - 1) / per_block) * per_block);
        const double balance = deal ? (double)n_g / (double)(((n_g + 7) / 8) * 8) : 1.0;
        if (fill * balance > best * 1.03) { best = fill * balance; group = g; }
    }
    const long long groups = (d.N + group - 1) / group;
    const long long bx = (group * EF + per_block - 1) / per_block;
    // one-dimensional grid: 8 XCDs x (groups per XCD) x M x blocks of positions
    const long long blocks = (deal ? 8 * ((groups + 7) / 8) : groups) * bx * ((d.M + rows - 1) / rows);
    if (blocks > 0x7FFFFFFFll || bx * d.M > 0x7FFFFFFFll) return ESCOIN_ERANGE;
    return launch(four ? sconv_direct_kernel<4, 8, 4> : sconv_direct_kernel<1, 16, 1>, dim3((unsigned)blocks), dim3(64 * rows), 0,
                  stream, d_rowptr, d_colidx, d_value, d_padded, d_out, d_bias, flags, d.N, d.M, d.E, d.F, d.Wp, (int)pitch,
                  d.stride, (int)img_elems, (int)group, (int)groups, (int)bx, (int)deal);
}

}  // namespace escoin

extern "C" int escoin_sconv_forward(const escoin_conv_desc* desc, const int32_t* d_rowptr,
                                    const int32_t* d_colidx_stretched, const float* d_value,
                                    const float* d_padded, float* d_out, const float* d_bias,
                                    uint32_t flags, void* hip_stream) {
    escoin::Dims d;
    int rc = escoin::make_dims(desc, &d);
    if (rc != ESCOIN_OK) return rc;
    if (!d_rowptr || !d_padded || !d_out) return ESCOIN_EINVAL;
    if (flags & ~(uint32_t)(ESCOIN_F_BIAS | ESCOIN_F_RELU)) return ESCOIN_EINVAL;
    if ((flags & ESCOIN_F_BIAS) && !d_bias) return ESCOIN_EINVAL;
    return escoin::launch_sconv_direct(d, d_rowptr, d_colidx_stretched, d_value, d_padded, d_out,
                                       d_bias, flags, (hipStream_t)hip_stream);
}
