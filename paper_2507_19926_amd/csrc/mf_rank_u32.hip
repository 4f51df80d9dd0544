// Ranked sliding-histogram kernels of 32-bit data: windows of up to 31 columns
// take up to 31 rows, wider ones are square. The batched kernels are those of
// the square windows that the library's own choice gives to this form.
#include "mf_rank_kernel.h"

bool mf_rank_kernel_u32(int kw, HistKernelInfo* k)
{
    switch (kw) {
    case 3: *k = rank_kernel<3, 31, uint32_t, false>(); return true;
    case 5: *k = rank_kernel<5, 31, uint32_t, false>(); return true;
    case 7: *k = rank_kernel<7, 31, uint32_t, false>(); return true;
    case 9: *k = rank_kernel<9, 31, uint32_t, false>(); return true;
    case 11: *k = rank_kernel<11, 31, uint32_t, false>(); return true;
    case 13: *k = rank_kernel<13, 31, uint32_t, false>(); return true;
    case 15: *k = rank_kernel<15, 31, uint32_t, false>(); return true;
    case 17: *k = rank_kernel<17, 31, uint32_t, false>(); return true;
    case 19: *k = rank_kernel<19, 31, uint32_t, false>(); return true;
    case 21: *k = rank_kernel<21, 31, uint32_t, true>(); return true;
    case 23: *k = rank_kernel<23, 31, uint32_t, true>(); return true;
    case 25: *k = rank_kernel<25, 31, uint32_t, true>(); return true;
    case 27: *k = rank_kernel<27, 31, uint32_t, true>(); return true;
    case 29: *k = rank_kernel<29, 31, uint32_t, true>(); return true;
    case 31: *k = rank_kernel<31, 31, uint32_t, true>(); return true;
    case 33: *k = rank_kernel<33, 33, uint32_t, true>(); return true;
    case 35: *k = rank_kernel<35, 35, uint32_t, true>(); return true;
    case 37: *k = rank_kernel<37, 37, uint32_t, true>(); return true;
    case 39: *k = rank_kernel<39, 39, uint32_t, true>(); return true;
    case 41: *k = rank_kernel<41, 41, uint32_t, true>(); return true;
    case 43: *k = rank_kernel<43, 43, uint32_t, true>(); return true;
    case 45: *k = rank_kernel<45, 45, uint32_t, true>(); return true;
    case 47: *k = rank_kernel<47, 47, uint32_t, true>(); return true;
    case 49: *k = rank_kernel<49, 49, uint32_t, true>(); return true;
    case 51: *k = rank_kernel<51, 51, uint32_t, true>(); return true;
    case 53: *k = rank_kernel<53, 53, uint32_t, true>(); return true;
    case 55: *k = rank_kernel<55, 55, uint32_t, true>(); return true;
    case 57: *k = rank_kernel<57, 57, uint32_t, true>(); return true;
    case 59: *k = rank_kernel<59, 59, uint32_t, true>(); return true;
    case 61: *k = rank_kernel<61, 61, uint32_t, true>(); return true;
    case 63: *k = rank_kernel<63, 63, uint32_t, true>(); return true;
    case 65: *k = rank_kernel<65, 65, uint32_t, true>(); return true;
    case 67: *k = rank_kernel<67, 67, uint32_t, true>(); return true;
    case 69: *k = rank_kernel<69, 69, uint32_t, true>(); return true;
    case 71: *k = rank_kernel<71, 71, uint32_t, true>(); return true;
    case 73: *k = rank_kernel<73, 73, uint32_t, true>(); return true;
    case 75: *k = rank_kernel<75, 75, uint32_t, true>(); return true;
    default: return false;
    }
}
