// Sliding-histogram forms of the median filter (mf_hist.hip): 8-bit planes
// (mf_hist_kernel.h), and 16- and 32-bit planes whose values are replaced by
// buckets of their ranks (mf_rank_kernel.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mf_internal.h"

// Form number of the data-aware variant in mf_options.
constexpr int kDaFormHist = 3;

// Everything the host needs of one window's kernels.
struct HistKernelInfo {
    const void* planes;
    const void* batched;    // null where no square window uses it
    int threads, cols, rows;   // output columns of a work-group; rows of a batched block
    size_t lds;
    // ranked kernels: most output rows of a region; those beyond `rows` run the
    // tall kernel
    int max_rows = 0;
    const void* tall = nullptr;
    size_t tall_lds = 0;
};

// Whether the kw x kh window (kw columns, kh rows, both odd) has a kernel.
bool mf_hist_supports(int dtype, int kw, int kh);
// `planes` planes of H x W, plane p at src/dst + p * plane_stride bytes.
hipError_t mf_hist_launch(const void* src, void* dst, int planes, long long plane_stride, int H, int W,
                          long long pitch, int dtype, int kw, int kh, hipStream_t stream);
// Estimated time in us of mf_hist_launch on the current device, good to a
// quarter, and that device's CUs; 0 where either is not known.
double mf_hist_estimate(int dtype, int kw, int kh, long long planes, int H, int W, int* cus);
// The same of an image's part in a batch, on 256 CUs.
double mf_hist_batched_estimate(int dtype, int k, int H, int W);
// Batched kernel of the square k x k window (arguments: jobs, njobs, nblocks).
hipError_t mf_hist_batched(int dtype, int k, MfBatchedKernel* kern);

// 3-D boxes, cubic k x k x k, of a D x H x W volume (rows pitch bytes apart,
// slices slice bytes).
bool mf_hist3_supports(int dtype, int k);
double mf_hist3_estimate(int D, int H, int W, int k, int* cus);     // us, as mf_hist_estimate
hipError_t mf_hist3_launch(const void* src, void* dst, int D, int H, int W, long long pitch, long long slice, int k,
                           hipStream_t stream);
