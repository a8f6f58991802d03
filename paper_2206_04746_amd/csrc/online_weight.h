// What the online trainers' translation units share (online.hip, online_batched.hip, online_chain.hip).
#pragma once

#include "hdc_internal.h"

namespace hdc {

// One record per sample, written by the step that takes the decisions, read by the one that
// updates the rows.
struct OnlineWeight {
    int32_t y;      // label, or -1: sample skipped
    int32_t pred;   // predicted class if it differs from y, else -1
    float w_y;      // float(1 - cos_y)
    float w_p;      // float(lr * (1 - cos_pred))
};

// A context-owned buffer of at least `want` bytes; a no-op when it is that large already.
template <typename T>
int grow(T **p, size_t *have, size_t want) {
    if (*have >= want) return HDC_OK;
    if (*p) HDC_HIP(hipFree(*p));   // waits for the device: nothing still reads the old buffer
    *p = nullptr;
    *have = 0;
    const hipError_t e = hipMalloc(reinterpret_cast<void **>(p), want + 256);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        return HDC_ENOMEM;
    }
    HDC_HIP(e);
    *have = want;
    return HDC_OK;
}

// Squared-norm partials of the rows into ob_norm_d (online_batched.hip).
int launch_norm(hdc_ctx_impl *c, const float *acc, int G, hipStream_t s);

// The block-wise walk of the chain (online_chain.hip): models it takes, batch sizes at which it is the
// faster way, its scratch (with the words of online_lds_kernel), the call (per_sample: hdc_train_online's
// arithmetic, else hdc_train_online_batched's).
constexpr int64_t kOnlineWords = 14 * 1024;   // samples x threads whose bit words online_lds_kernel is handed (56 KB)
bool online_chain_takes(const hdc_ctx_impl *c);
bool online_chain_pays(const hdc_ctx_impl *c, int64_t N, int64_t batch);
int reserve_online_chain(hdc_ctx_impl *c);
int reserve_online_blocks(hdc_ctx_impl *c);   // without that of longer blocks (online_spread.hip)
// Whether a call may go in blocks: a model they take, their scratch there or to be had.  False without an
// error (*rc HDC_OK) while the stream is captured or memory is short: such a call goes another way.
bool online_chain_ready(hdc_ctx_impl *c, hipStream_t s, int *rc);
int launch_online_chain(hdc_ctx_impl *c, const uint32_t *hv, const int32_t *labels, int64_t N, int32_t epochs,
                        float lr, int64_t batch, bool per_sample, float *acc, hipStream_t s);


// Partial dot products of nb samples with the rows (row_dots.hip), part[slice * stride + n * step_n + class * step_c], and, where
// normpart is given, the rows' squared-norm partials.  *slices: how many there are, row_dots_slices at most.
int row_dots_slices(int D, int most);
int launch_row_dots(hdc_ctx_impl *c, const uint32_t *hv, int64_t nb, const float *acc, double *part, int64_t stride, int64_t step_n,
                    int64_t step_c, double *normpart, int most, int *slices, hipStream_t s);

// Calls of many samples in blocks of kSpan, each block's chain spread over kSpan / kStripCols workgroups
// (online_spread.hip).
constexpr int kSpan = 2048;         // most samples of a block
constexpr int kStripCols = 16;      // samples of a workgroup
// Products of a block's samples: strip after strip of 16 columns, of each the rows of the samples up to its last one.
__host__ __device__ constexpr int strip_start(int strip) { return kStripCols * kStripCols * strip * (strip + 1) / 2; }
constexpr int kSpanProducts = strip_start(kSpan / kStripCols);
bool online_spread_pays(const hdc_ctx_impl *c, int64_t N, int64_t batch);   // in batches: worth asking for scratch
bool online_spread_takes(const hdc_ctx_impl *c, int64_t N, float lr, int64_t batch, bool per_sample);
int reserve_online_spread(hdc_ctx_impl *c);
template <bool BATCH>
int launch_online_spread(hdc_ctx_impl *c, const uint32_t *hv, const int32_t *labels, int64_t N, int32_t epochs, float lr,
                         int batch, float *acc, hipStream_t s);

// Steps of both forms of the block-wise walk (online_chain.hip): the samples' bits by dimension groups (col[group][ld])
// and the products of a block's samples in strips.
int64_t held_samples(int G);
void launch_columns(hdc_ctx_impl *c, const uint32_t *hv, int64_t n, int64_t ld, hipStream_t s);
void launch_strips(hdc_ctx_impl *c, int64_t n, int64_t ld, int block, int16_t *strips, hipStream_t s);

}  // namespace hdc
