// Sliding-histogram kernels of the 3-D boxes: the 9 values of a column of the
// 3 x 3 x 3 box fit the one-word layout's four bits, larger boxes take two
// words (at most 225 values to a column).
#include "mf_hist_kernel.h"

bool mf_hist_kernel_box(int k, HistKernelInfo* h)
{
    switch (k) {
    case 3: *h = hist3_kernel<3, 1>(); return true;
    case 5: *h = hist3_kernel<5, 2>(); return true;
    case 7: *h = hist3_kernel<7, 2>(); return true;
    case 9: *h = hist3_kernel<9, 2>(); return true;
    case 11: *h = hist3_kernel<11, 2>(); return true;
    case 13: *h = hist3_kernel<13, 2>(); return true;
    case 15: *h = hist3_kernel<15, 2>(); return true;
    default: return false;
    }
}
