// Sliding-histogram kernels: one counter word, windows up to 31 columns of which
// some have no network. The batched kernels are those of the square windows that
// the library's own choice gives to this form.
#include "mf_hist_kernel.h"

bool mf_hist_kernel_p1(int kw, HistKernelInfo* k)
{
    switch (kw) {
    case 9: *k = hist_kernel<9, 1, false>(); return true;
    case 11: *k = hist_kernel<11, 1, false>(); return true;
    case 13: *k = hist_kernel<13, 1, true>(); return true;
    case 15: *k = hist_kernel<15, 1, true>(); return true;
    case 19: *k = hist_kernel<19, 1, false>(); return true;
    case 21: *k = hist_kernel<21, 1, false>(); return true;
    case 23: *k = hist_kernel<23, 1, false>(); return true;
    case 25: *k = hist_kernel<25, 1, false>(); return true;
    case 27: *k = hist_kernel<27, 1, false>(); return true;
    case 29: *k = hist_kernel<29, 1, false>(); return true;
    default: return false;
    }
}
