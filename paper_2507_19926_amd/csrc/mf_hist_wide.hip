// Sliding-histogram kernels: two counter words, windows of 33 to 75 columns. The batched kernels
// are those of the square windows that the library's own choice gives to
// this form.
#include "mf_hist_kernel.h"

bool mf_hist_kernel_wide(int kw, HistKernelInfo* k)
{
    switch (kw) {
    case 33: *k = hist_kernel<33, 2, true>(); return true;
    case 35: *k = hist_kernel<35, 2, true>(); return true;
    case 37: *k = hist_kernel<37, 2, true>(); return true;
    case 39: *k = hist_kernel<39, 2, true>(); return true;
    case 41: *k = hist_kernel<41, 2, true>(); return true;
    case 43: *k = hist_kernel<43, 2, true>(); return true;
    case 45: *k = hist_kernel<45, 2, true>(); return true;
    case 47: *k = hist_kernel<47, 2, true>(); return true;
    case 49: *k = hist_kernel<49, 2, true>(); return true;
    case 51: *k = hist_kernel<51, 2, true>(); return true;
    case 53: *k = hist_kernel<53, 2, true>(); return true;
    case 55: *k = hist_kernel<55, 2, true>(); return true;
    case 57: *k = hist_kernel<57, 2, true>(); return true;
    case 59: *k = hist_kernel<59, 2, true>(); return true;
    case 61: *k = hist_kernel<61, 2, true>(); return true;
    case 63: *k = hist_kernel<63, 2, true>(); return true;
    case 65: *k = hist_kernel<65, 2, true>(); return true;
    case 67: *k = hist_kernel<67, 2, true>(); return true;
    case 69: *k = hist_kernel<69, 2, true>(); return true;
    case 71: *k = hist_kernel<71, 2, true>(); return true;
    case 73: *k = hist_kernel<73, 2, true>(); return true;
    case 75: *k = hist_kernel<75, 2, true>(); return true;
    default: return false;
    }
}
