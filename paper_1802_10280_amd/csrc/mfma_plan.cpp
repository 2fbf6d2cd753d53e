// Host side of the matrix-core form: which layers have one, and its section of the plan.
#include <math.h>
#include <string.h>

#include <vector>

#include "mfma.h"

namespace escoin {

// Microseconds for a batch of N images, and whether that is faster than the tiled kernel.  A workgroup alone on its compute unit spends 1.6 us on a chunk (staging, barrier, the first
// wait) and 0.46 us on each of its taps; two that share one take 1.72 times as long for both.  The tiled
// kernel is taken at its better: 36 TFLOP/s on the nonzeros (41 measured on a large layer at 50 % sparsity, 32
// on 13x13 maps at 65 %, less the fewer nonzeros or positions there are).
// Windows above kMfmaPairWindow leave no LDS for a second workgroup: rounds are of 256, each as long as one.
// That is 57.9, 86.9, 115.8 and 332 us where 56-58, 85, 115 and 341 were measured (64 channels, 25, 35 and 62
// images of 63x63; 128 channels, 5x5, 64 of 32x32), so the margin can go; on such layers the tiled kernel was
// 4-25 % slower than its estimate (67, 118, 158, 393 us at 71-75 and 65 % sparsity).
double mfma_time(const Dims& d, double N) {
    const double jobs = ceil(N * (d.H + d.pad) * (d.W + d.pad) / kMfmaTP) * (double)(mfma_row_blocks(d) / kMfmaWM);
    const double job = 6.0 + (double)mfma_chunks(d) * (1.6 + 0.46 * d.R * d.S);
    if (jobs <= 256) return job;
    if (mfma_window(d) <= kMfmaPairWindow) return ceil(jobs / 512) * 1.72 * job;
    return ceil(jobs / 256) * job;
}
static bool mfma_faster(const Dims& d, double N, long long nnz) {
    const double jobs = ceil(N * (d.H + d.pad) * (d.W + d.pad) / kMfmaTP) * (double)(mfma_row_blocks(d) / kMfmaWM);
    const double tiled = 2e-6 * (double)nnz * N * d.E * d.F / 36.0;
    return mfma_time(d, N) < (jobs <= 256 || mfma_window(d) <= kMfmaPairWindow ? 0.9 : 1.04) * tiled;
}

// Whether a plan carries the section: shapes the kernel takes, and pruned so little that a batch that
// suits it is faster on the matrix cores: one of many workgroups, or of two full rounds where they do not pair.
bool mfma_planned(const Dims& d, long long nnz) {
    if (d.stride != 1 || d.R <= d.pad || d.S <= d.pad || mfma_window(d) > kMfmaMaxWindow) return false;
    if (d.C < 16 || d.M < 32 || mfma_weight_bytes(d) > (64ull << 20)) return false;
    const double groups = (double)(mfma_row_blocks(d) / kMfmaWM);
    const double tiles = mfma_window(d) <= kMfmaPairWindow ? 512.0 * 64 : floor(512.0 / groups);
    return mfma_faster(d, tiles * kMfmaTP / ((double)(d.H + d.pad) * (d.W + d.pad)), nnz);
}

// Whether a forward call on this batch takes the section of a plan made for this layer: offsets inside the
// kernel are 32 bits, and the batch has to fill the compute units.
bool mfma_taken(const Dims& d, const PlanHeader& h) {
    if (h.mfma != 1 || h.mfma_nnz <= 0 || !mfma_planned(d, h.mfma_nnz)) return false;
    const long long total = (long long)d.N * (d.H + d.pad) * (d.W + d.pad);
    const long long groups = (long long)mfma_row_blocks(d) / kMfmaWM;
    if (total > (1ll << 30) || (long long)d.N * d.C * d.H * d.W > (1ll << 30) || total / kMfmaTP * groups > (1ll << 30)) return false;
    return mfma_faster(d, d.N, h.mfma_nnz);
}

static float to_bf16(float x, uint16_t* bits) {  // rounds to nearest even; x is finite
    uint32_t u;
    memcpy(&u, &x, 4);
    u = (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
    *bits = (uint16_t)(u >> 16);
    float r;
    memcpy(&r, &u, 4);
    return r;
}

// Writes the row pointers and the nonzero values, decoded, into `out`.  False where a column is repeated: its
// values would have to be added up first.
bool nz_write(const Dims& d, const int32_t* rowptr, const int32_t* stretched, const float* value, char* out) {
    const size_t RS = (size_t)d.R * d.S;
    int32_t* rp = (int32_t*)out;
    MfmaNz* nz = (MfmaNz*)(out + mfma_rowptr_bytes(d));
    std::vector<int32_t> seen((size_t)d.C * RS, -1);
    const int32_t plane = d.Hp * d.Wp;
    int32_t at = 0;
    for (int m = 0; m < d.M; ++m) {
        rp[m] = at;
        for (int j = rowptr[m]; j < rowptr[m + 1]; ++j) {
            if (value[j] == 0.0f) continue;
            const int c = stretched[j] / plane, rem = stretched[j] - c * plane, r = rem / d.Wp, s = rem - r * d.Wp;
            int32_t& was = seen[(size_t)c * RS + (size_t)r * d.S + s];
            if (was == m) return false;
            was = m;
            nz[at].c = c;
            nz[at].r = (uint16_t)r;
            nz[at].s = (uint16_t)s;
            nz[at].val = value[j];
            ++at;
        }
    }
    rp[d.M] = at;
    return true;
}

// Writes the split weights into `out` (zeroed).  False where one is outside the range whose split keeps fp32
// (Inf and NaN too).
bool mfma_write(const Dims& d, const int32_t* rp, const MfmaNz* nz, char* out) {
    const size_t RS = (size_t)d.R * d.S, chunks = mfma_chunks(d);
    uint16_t* w = (uint16_t*)out;
    for (int m = 0; m < d.M; ++m)
        for (int j = rp[m]; j < rp[m + 1]; ++j) {
            const float v = nz[j].val;
            const int c = nz[j].c;
            uint16_t part[3];
            if (!(fabsf(v) >= kMfmaLeastWeight && fabsf(v) <= kMfmaMostWeight)) return false;
            const float rest = v - to_bf16(v, &part[0]);
            to_bf16(rest - to_bf16(rest, &part[1]), &part[2]);
            // lane: channel m % 32, and which 8 of the 16 input channels; 8 of them per lane
            const size_t step = ((size_t)(m / 32) * chunks + c / 16) * RS + (size_t)nz[j].r * d.S + nz[j].s;
            const size_t lane = m % 32 + 32 * (size_t)(c % 16 / 8);
            for (int k = 0; k < 3; ++k) w[((step * 3 + k) * 64 + lane) * 8 + c % 8] = part[k];
        }
    return true;
}

}  // namespace escoin
