// Sliding-histogram kernels: two counter words, windows up to 31 columns. The batched kernels
// are those of the square windows that the library's own choice gives to
// this form.
#include "mf_hist_kernel.h"

bool mf_hist_kernel_p2(int kw, HistKernelInfo* k)
{
    switch (kw) {
    case 3: *k = hist_kernel<3, 2, false>(); return true;
    case 5: *k = hist_kernel<5, 2, false>(); return true;
    case 7: *k = hist_kernel<7, 2, false>(); return true;
    case 9: *k = hist_kernel<9, 2, false>(); return true;
    case 11: *k = hist_kernel<11, 2, false>(); return true;
    case 13: *k = hist_kernel<13, 2, false>(); return true;
    case 15: *k = hist_kernel<15, 2, false>(); return true;
    case 17: *k = hist_kernel<17, 2, true>(); return true;
    case 19: *k = hist_kernel<19, 2, true>(); return true;
    case 21: *k = hist_kernel<21, 2, true>(); return true;
    case 23: *k = hist_kernel<23, 2, true>(); return true;
    case 25: *k = hist_kernel<25, 2, true>(); return true;
    case 27: *k = hist_kernel<27, 2, true>(); return true;
    case 29: *k = hist_kernel<29, 2, true>(); return true;
    case 31: *k = hist_kernel<31, 2, true>(); return true;
    default: return false;
    }
}
