// The matrix-core form of the layer: what its plan section holds and which layers have one.
#pragma once
#include "common.h"
#include "plan.h"

namespace escoin {

constexpr int kMfmaWM = 2, kMfmaWP = 4;      // waves of a workgroup over channels (32 each) and positions (64 each)
constexpr int kMfmaTP = 64 * kMfmaWP;        // output positions of a workgroup
constexpr int kMfmaMaxWindow = 512;          // window positions it can stage (two tasks a thread)
constexpr int kMfmaPairWindow = 384;         // up to here two workgroups fit the LDS of a compute unit

// The weights the section can hold.  Below 2^-110 the three bf16 parts are no longer exact (bf16 ends at
// 2^-133, fp32 at 2^-149).  The limits lie well inside that, so that the products keep their bits with
// inputs down to 2^-70 (the kernel looks for smaller ones).
constexpr float kMfmaLeastWeight = 0x1p-50f, kMfmaMostWeight = 0x1p30f;

// A nonzero, for the outputs whose sums cannot be used.
struct MfmaNz {
    int32_t c;
    uint16_t r, s;
    float val;
};

// window positions a workgroup reads: its own and the reach of the taps
inline long long mfma_window(const Dims& d) {
    return kMfmaTP + (long long)(d.R - 1) * (d.W + d.pad) + d.S - 1;
}
inline uint64_t mfma_row_blocks(const Dims& d) { return (uint64_t)(d.M + 32 * kMfmaWM - 1) / (32 * kMfmaWM) * kMfmaWM; }
inline uint64_t mfma_chunks(const Dims& d) { return ((uint64_t)d.C + 15) / 16; }
// three splits of 1024 bytes per (32 channels, 16 input channels, tap), and one step to read ahead
inline uint64_t mfma_weight_bytes(const Dims& d) {
    return (mfma_row_blocks(d) * mfma_chunks(d) * d.R * d.S + 1) * 3072;
}
inline uint64_t mfma_rowptr_bytes(const Dims& d) { return ((uint64_t)(d.M + 1) * 4 + 255) / 256 * 256; }
inline uint64_t nz_bytes(const Dims& d, int nnz) { return mfma_rowptr_bytes(d) + (uint64_t)nnz * sizeof(MfmaNz); }

double mfma_time(const Dims& d, double N);
bool mfma_planned(const Dims& d, long long nnz);
bool mfma_taken(const Dims& d, const PlanHeader& h);
bool nz_write(const Dims& d, const int32_t* rowptr, const int32_t* stretched, const float* value, char* out);
bool mfma_write(const Dims& d, const int32_t* rp, const MfmaNz* nz, char* out);
int launch_sconv_mfma(const Dims& d, const PlanHeader& h, const char* d_plan, const float* d_in, float* d_out,
                      const float* d_bias, uint32_t flags, hipStream_t stream);
int allow_dynamic_lds(const void* kernel, int bytes);

}  // namespace escoin
