// Sliding-histogram forms: choice of kernel and launch (the kernels are
// described in mf_hist_kernel.h and mf_rank_kernel.h).
#include <atomic>

#include "mf_hist_kernel.h"

// P = 1 and P = 2 kernels of the windows up to 31 columns, P = 2 from 33 on
// (mf_hist_p1.hip, mf_hist_p2.hip, mf_hist_wide.hip).
bool mf_hist_kernel_p1(int kw, HistKernelInfo* k);
bool mf_hist_kernel_p2(int kw, HistKernelInfo* k);
bool mf_hist_kernel_wide(int kw, HistKernelInfo* k);
// 16- and 32-bit data (mf_rank_u16.hip, mf_rank_u32.hip)
bool mf_rank_kernel_u16(int kw, HistKernelInfo* k);
bool mf_rank_kernel_u32(int kw, HistKernelInfo* k);
// 3-D boxes (mf_hist_box.hip)
bool mf_hist_kernel_box(int k, HistKernelInfo* h);

namespace {

constexpr int kMaxDevices = 64;
constexpr int kTallSlots = 8 * 38 + 16;   // slot_of() of windows, boxes, then tall ranked kernels
constexpr int kSlots = kTallSlots + 38;

// All counts of the window fit the one-word layout: 4 bits for a column's
// kh values, 8 for the kw - 3 shared columns'.
bool one_word(int kw, int kh) { return kh <= 15 && kh * (kw - 3) <= 255; }

bool find(int dtype, int kw, int kh, HistKernelInfo* k)
{
    if (kw < 3 || kw % 2 == 0 || kh < 1) return false;
    if (dtype != MF_U8) {
        if (kw <= 31 ? kh > 31 : kh != kw) return false;
        return dtype == MF_U16 ? mf_rank_kernel_u16(kw, k) : mf_rank_kernel_u32(kw, k);
    }
    if (kh > 255) return false;
    if (one_word(kw, kh) && mf_hist_kernel_p1(kw, k)) return true;
    return kw <= 31 ? mf_hist_kernel_p2(kw, k) : mf_hist_kernel_wide(kw, k);
}

// The kernels take more than 64 KB of LDS, which has to be allowed once per
// device and kernel.
hipError_t allow_lds(const void* fn, int slot, int dev)
{
    static std::atomic<unsigned char> done[kMaxDevices][kSlots];
    if (done[dev][slot].load(std::memory_order_acquire)) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess) done[dev][slot].store(1, std::memory_order_release);
    return e;
}

hipError_t device(int* dev, int* cus)
{
    static std::atomic<int> count[kMaxDevices];
    hipError_t e = hipGetDevice(dev);
    if (e != hipSuccess) return e;
    if (*dev < 0 || *dev >= kMaxDevices) return hipErrorInvalidDevice;
    *cus = count[*dev].load(std::memory_order_relaxed);
    if (*cus == 0) {
        e = hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, *dev);
        if (e != hipSuccess) return e;
        count[*dev].store(*cus, std::memory_order_relaxed);
    }
    return hipSuccess;
}

// Rows of a strip, for `per_strip` work-groups side by side: a strip costs its
// rows and `first` more for its first window; two work-groups run on each CU,
// so of the launches of r rounds the one that fills them is the cheapest.
// steps: row steps of the longest CU.
// rounds: strips of a work-group's place.
int strip_rows(int H, long long per_strip, long long first, int cus, long long* steps = nullptr, long long* rounds = nullptr)
{
    const long long slots = 2LL * cus;
    long long best = -1;
    int R = H;
    for (int r = 1; r <= 8; ++r) {
        long long n = r * slots / per_strip;
        if (n < 1) n = 1;
        if (n > H) n = H;
        const int rows = (int)((H + n - 1) / n);
        const long long strips = (H + rows - 1) / rows;
        const long long cost = ((strips * per_strip + slots - 1) / slots) * (rows + first);
        if (best < 0 || cost < best) {
            best = cost, R = rows;
            if (rounds) *rounds = (strips * per_strip + slots - 1) / slots;
        }
    }
    if (steps) *steps = best;
    return R;
}

// Output rows of a ranked region, by the measured clocks of its parts (uniform
// noise, k = 25..75): 4 (16-bit), 9 (32-bit) or 12 (32-bit, tall kernel) for a
// value of the footprint, loaded, sorted and listed, 300 for a row of the first
// window, 1600 for an output row slid, searched and walked; one region to a CU.
// clocks, rounds: of all regions of a CU.
int rank_rows(int H, int max_rows, long long per_strip, int fw, int kh, bool wide, int cus, long long* clocks = nullptr,
              long long* rounds = nullptr)
{
    long long best = -1;
    int R = max_rows;
    for (int r = max_rows; r >= 8; r -= 8) {
        const long long regions = (H + r - 1) / r * per_strip;
        const int used = r < H ? r : H;
        const long long value = !wide ? 4 : r <= 64 ? 9 : 12;
        const long long cost = (regions + cus - 1) / cus *
                               (value * fw * (used + kh - 1) + 300LL * kh + 1600LL * used + 5000);
        if (best < 0 || cost < best) {
            best = cost, R = r;
            if (rounds) *rounds = (regions + cus - 1) / cus;
        }
    }
    if (clocks) *clocks = best;
    return R;
}

// one number for each kernel of a window
int slot_of(int dtype, int kw, int kh, bool batched)
{
    const int kind = dtype == MF_U16 ? 2 : dtype != MF_U8 ? 3 : one_word(kw, kh) && kw <= 31 ? 0 : 1;
    return (kw / 2) * 8 + kind * 2 + (batched ? 1 : 0);
}

}  // namespace

bool mf_hist_supports(int dtype, int kw, int kh)
{
    HistKernelInfo k;
    return find(dtype, kw, kh, &k);
}

hipError_t mf_hist_launch(const void* src, void* dst, int planes, long long plane_stride, int H, int W,
                          long long pitch, int dtype, int kw, int kh, hipStream_t stream)
{
    HistKernelInfo k;
    if (!find(dtype, kw, kh, &k)) return hipErrorInvalidValue;
    int dev = 0, cus = 0;
    hipError_t e = device(&dev, &cus);
    if (e != hipSuccess) return e;
    const int ncol = (W + k.cols - 1) / k.cols;
    const bool rank = dtype != MF_U8;
    const int R = rank ? rank_rows(H, k.max_rows, (long long)ncol * planes, k.cols + kw - 1, kh, dtype != MF_U16, cus)
                       : strip_rows(H, (long long)ncol * planes, kh / 4 + 8, cus);
    int is_float = dtype == MF_F32;
    const bool tall = rank && R > k.rows;
    const void* fn = tall ? k.tall : k.planes;
    const size_t lds = tall ? k.tall_lds : k.lds;
    e = allow_lds(fn, tall ? kTallSlots + kw / 2 : slot_of(dtype, kw, kh, false), dev);
    if (e != hipSuccess) return e;
    const int ns = (H + R - 1) / R;
    const long long blocks = (long long)ncol * ns;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    // a grid has fewer than 2^32 threads a row: 2^23 - 1 regions of the ranked
    // kernels, the others' strips never come to so many
    const long long most = rank ? ((1LL << 32) - 1) / k.threads : blocks;
    for (int p0 = 0; p0 < planes; p0 += 65535) {     // grid rows are planes
        const int np = planes - p0 < 65535 ? planes - p0 : 65535;
        const unsigned char* s8 = (const unsigned char*)src + p0 * plane_stride;
        unsigned char* d8 = (unsigned char*)dst + p0 * plane_stride;
        for (long long from = 0; from < blocks; from += most) {
            int b0 = (int)from;
            const long long nb = blocks - from < most ? blocks - from : most;
            void* args[] = {&s8,         &d8,       &H,  &W,        &pitch, &plane_stride,
                            (void*)&ncol, (void*)&R, &kh, &is_float, &b0};     // the last two: ranked kernels
            e = hipLaunchKernel(fn, dim3((unsigned)nb, np), dim3(k.threads), args, lds, stream);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

// 8-bit: 8 us and the row steps (noise, which takes longer than a smooth image,
// on many planes of 16 x 16: k = 23 0.62 us a step, 35 0.70, 75 1.1); ranked: 8 us,
// the clocks above and 12 us a round (float32 k = 25: 16 x 16 to a plane 3.0 / 3.5 us
// measured / estimated for 12 of them, 2048^2 200 / 182 us).
double mf_hist_estimate(int dtype, int kw, int kh, long long planes, int H, int W, int* cus)
{
    HistKernelInfo k;
    int dev = 0;
    if (!find(dtype, kw, kh, &k) || device(&dev, cus) != hipSuccess) return 0;
    const long long per_strip = planes * ((W + k.cols - 1) / k.cols);
    if (dtype == MF_U8) {
        long long steps = 0;
        strip_rows(H, per_strip, kh / 4 + 8, *cus, &steps);
        return 8 + (double)steps * (0.4 + 0.0096 * kw);
    }
    long long clocks = 0, rounds = 0;
    rank_rows(H, k.max_rows, per_strip, k.cols + kw - 1, kh, dtype != MF_U16, *cus, &clocks, &rounds);
    return 8 + (double)clocks / 2400 + 12.0 * (double)rounds;
}

double mf_hist_batched_estimate(int dtype, int k, int H, int W)
{
    HistKernelInfo h;
    if (!find(dtype, k, k, &h)) return 0;
    const double blocks = (double)((W + h.cols - 1) / h.cols) * ((H + h.rows - 1) / h.rows);
    const int used = H < h.rows ? H : h.rows;
    if (dtype == MF_U8) return blocks / 512 * (used + k / 4 + 8) * (0.4 + 0.0096 * k);
    const double clocks = (dtype == MF_U16 ? 4.0 : 9.0) * (h.cols + k - 1) * (used + k - 1) + 300.0 * k + 1600.0 * used + 5000;
    return blocks / 256 * (clocks / 2400 + 12);
}

hipError_t mf_hist_batched(int dtype, int k, MfBatchedKernel* kern)
{
    HistKernelInfo h;
    if (!find(dtype, k, k, &h) || !h.batched) return hipErrorInvalidValue;
    int dev = 0, cus = 0;
    hipError_t e = device(&dev, &cus);
    if (e != hipSuccess) return e;
    e = allow_lds(h.batched, slot_of(dtype, k, k, true), dev);
    if (e != hipSuccess) return e;
    kern->fn = h.batched;
    kern->threads = h.threads;
    kern->lds = h.lds;
    kern->bw = h.cols;
    kern->bh = h.rows;
    return hipSuccess;
}

bool mf_hist3_supports(int dtype, int k)
{
    HistKernelInfo h;
    return dtype == MF_U8 && mf_hist_kernel_box(k, &h);
}

// 8 us, and in each round the first window and the row steps (128 x 128 x 128 of
// noise, measured / estimated: k = 5 58 / 66 us, 9 77 / 106, 15 255 / 254; 128 x 4 x 32
// k = 15 85 / 91).
double mf_hist3_estimate(int D, int H, int W, int k, int* cus)
{
    HistKernelInfo h;
    int dev = 0;
    if (!mf_hist_kernel_box(k, &h) || device(&dev, cus) != hipSuccess) return 0;
    const int first = k * k / 4 + 8;
    long long rounds = 0;
    const int R = strip_rows(H, (long long)((W + h.cols - 1) / h.cols) * D, first, *cus, nullptr, &rounds);
    return 8 + (double)rounds * ((0.2 + 0.0045 * k * k) * first + (1.2 + 0.018 * k * k) * R);
}

hipError_t mf_hist3_launch(const void* src, void* dst, int D, int H, int W, long long pitch, long long slice, int k,
                           hipStream_t stream)
{
    HistKernelInfo h;
    if (!mf_hist_kernel_box(k, &h)) return hipErrorInvalidValue;
    int dev = 0, cus = 0;
    hipError_t e = device(&dev, &cus);
    if (e != hipSuccess) return e;
    e = allow_lds(h.planes, 8 * 38 + k, dev);
    if (e != hipSuccess) return e;
    const int ncol = (W + h.cols - 1) / h.cols;
    const int R = strip_rows(H, (long long)ncol * D, k * k / 4 + 8, cus);
    const int ns = (H + R - 1) / R;
    if ((long long)ncol * ns > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    for (int z0 = 0; z0 < D; z0 += 65535) {          // grid rows are slices
        const int nz = D - z0 < 65535 ? D - z0 : 65535;
        void* args[] = {&src, &dst, &D, &H, &W, &pitch, &slice, (void*)&ncol, (void*)&R, &z0};
        e = hipLaunchKernel(h.planes, dim3((unsigned)(ncol * ns), nz), dim3(h.threads), args, h.lds, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
