// Differentiable form of the median filter: argmedian in the forward pass and
// a deterministic gather in the backward pass. The paper has no gradients;
// the rules below are the library's.
//
// Forward: the median value comes from the hierarchical kernels; then each
// output pixel p scans its clamped k x k window in row-major order and
// records the plane-flat index of the first input pixel whose bits equal the
// median. Because clamping is monotone this is the lowest flat index among
// the window pixels holding the median.
//
// Backward: grad_in[q] = sum of grad_out[p] over output pixels p whose
// argmedian is q. Such p lie within r = (k-1)/2 of q in both directions, so
// each q gathers over its (2r+1)^2 neighbours in ascending flat order of p
// and adds in binary32 from +0. That is exactly the order of a scatter in
// ascending p, so the result is bit-reproducible and needs no atomics.
#include "mf_internal.h"

namespace {

constexpr int kBX = 64, kBY = 4;           // output block of one work-group
constexpr int kThreads = kBX * kBY;

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return min(max(v, lo), hi); }

}  // namespace

// One work-group: a 64 x 4 kRows block of one plane, kRows (four) output rows to
// a lane. The window union ((64 + k - 1) x (16 + k - 1) values) is staged in LDS as
// float bits; a row of it that lies in several of the lane's windows is read
// once and compared with each of their medians. The match of a whole row is
// one bit per lane, so a comparison is one VALU instruction (its or is
// scalar); the row found is then read again, from its end, for the column.
//
// Bound: VALU, 1.5 k * k instructions per output. 32x3x512x512: k = 7 0.31 ms with
// one row to a lane (k * k reads, compares and selects), 0.14 now; k = 15 0.75
// and 0.37. Where a wave's medians all lie in the first rows of their windows,
// as in images of few levels, the wave ends there: it looks once, after eight
// rows (with the median, two levels, us, a stop at the first match / none /
// now: 100 x 300 k = 33 28 / 58 / 31, 32 x 512 x 512 k = 15 243 / 296 / 245). Few blocks
// of a large window take one row to a lane, whose wave ends sooner (100 x 300 k = 25,
// with the median, noise 52 and 40 us). (A scalar or of the compares' masks
// instead of v_min3: k = 7 0.15, k = 15 1.31, the masks outgrow the scalar registers.)
template <int K, int kRows>
__global__ void __launch_bounds__(kThreads)
mf_argmedian_kernel(const uint32_t* __restrict__ src, const uint32_t* __restrict__ med,
                    int32_t* __restrict__ idx, int H, int W, int k_rt, int nbx, int nby)
{
    extern __shared__ uint32_t tile[];
    const int k = K ? K : k_rt;
    const int plane = blockIdx.x / (nbx * nby);
    const int b = blockIdx.x - plane * nbx * nby;
    const int by = b / nbx, bx = b - by * nbx;
    const int r = (k - 1) / 2;
    const long long base = (long long)plane * H * W;
    constexpr int kAY = kBY * kRows;
    const int X0 = bx * kBX, Y0 = by * kAY;
    const int lw = kBX + 2 * r, lh = kAY + 2 * r;
    for (int i = threadIdx.x; i < lw * lh; i += kThreads) {
        const int y = i / lw, x = i - y * lw;
        const int gy = clampi(Y0 - r + y, 0, H - 1), gx = clampi(X0 - r + x, 0, W - 1);
        tile[i] = src[base + (long long)gy * W + gx];
    }
    const int tx = threadIdx.x % kBX, ty = threadIdx.x / kBX * kRows;
    const int x = X0 + tx;
    uint32_t m[kRows];
    int row[kRows];            // first row of the window that holds the median
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int y = min(Y0 + ty + j, H - 1);
        m[j] = med[base + (long long)y * W + min(x, W - 1)];
        row[j] = x < W && Y0 + ty + j < H ? -1 : 0;
    }
    __syncthreads();
    if (Y0 + ty >= H) return;  // a whole wave
    auto scan = [&](int t) {
        const uint32_t* p = tile + (ty + t) * lw + tx;
        uint32_t off[kRows];   // 0 where the row holds the median
#pragma unroll
        for (int j = 0; j < kRows; ++j) off[j] = p[0] ^ m[j];
#pragma unroll 4
        for (int dx = 1; dx < k; dx += 2) {
            const uint32_t v = p[dx], u = p[dx + 1];
#pragma unroll
            for (int j = 0; j < kRows; ++j) off[j] = min(off[j], min(v ^ m[j], u ^ m[j]));
        }
#pragma unroll
        for (int j = 0; j < kRows; ++j)
            if (t >= j && t - j < k) row[j] = off[j] == 0 && row[j] < 0 ? t - j : row[j];
    };
    const int n = k + kRows - 1, look = k > 7 ? 8 : n;
    for (int t = 0; t < look; ++t) scan(t);
    int least = row[0];
#pragma unroll
    for (int j = 1; j < kRows; ++j) least = min(least, row[j]);
    if (!__all(least >= 0))
        for (int t = look; t < n; ++t) scan(t);
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int y = Y0 + ty + j;
        if (y >= H || x >= W) continue;
        const uint32_t* p = tile + (ty + j + max(row[j], 0)) * lw + tx;
        int col = 0;
#pragma unroll 8
        for (int dx = k - 1; dx >= 0; --dx) col = p[dx] == m[j] ? dx : col;
        idx[base + (long long)y * W + x] =
            row[j] < 0 ? -1 : clampi(y - r + row[j], 0, H - 1) * W + clampi(x - r + col, 0, W - 1);
    }
}

// Backward, windows of up to 31: a work-group takes 64 x ROWS input pixels. An
// output pixel p that names one of them, q, sets in q's bit map the bit of
// its place in q's window (rows of RB bits: 8, 16 or 32 for k up to 7, 15 and
// 31); bits are set by LDS or, in any order. Every q then adds grad_out over
// its set bits from the lowest on, which is ascending p. Work per pixel is one
// or and one addition per naming instead of k * k comparisons.
//
// Bound: instruction issue and LDS latency of the bit loops (a wave runs as
// long as its most named pixel), from k = 17 on the LDS the maps leave for
// other work-groups. 32x3x512x512, comparing k * k neighbours and now: k = 7
// 0.35 and 0.18 ms, k = 15 0.91 and 0.36, k = 31 3.8 and 0.99. Small windows of few
// pixels compare (k = 7, us: 100 x 300 7.2 against 9.3, 512 x 512 8.0 against 9.0).
template <int RB, int ROWS, int THREADS>
__global__ void __launch_bounds__(THREADS)
mf_grad_bits_kernel(const float* __restrict__ gout, const int32_t* __restrict__ idx, float* __restrict__ gin, int H,
                    int W, int k, int nbx, int nby, uint32_t inv_w, uint32_t inv_lw)
{
    extern __shared__ uint32_t bits[];       // [words][kBX * ROWS], then the grad_out tile
    constexpr int kQ = kBX * ROWS;
    const int words = (k * RB + 31) / 32;
    float* const g = reinterpret_cast<float*>(bits + words * kQ);
    const int plane = blockIdx.x / (nbx * nby);
    const int b = blockIdx.x - plane * nbx * nby;
    const int by = b / nbx, bx = b - by * nbx;
    const int r = (k - 1) / 2;
    const long long base = (long long)plane * H * W;
    const int X0 = bx * kBX, Y0 = by * ROWS;
    const int lw = kBX + 2 * r, lh = ROWS + 2 * r;
    for (int i = threadIdx.x; i < words * kQ; i += THREADS) bits[i] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < lw * lh; i += THREADS) {
        const int y = (int)((uint32_t)i * inv_lw >> 20), x = i - y * lw;    // i / lw for i < 2^12
        const int py = Y0 - r + y, px = X0 - r + x;
        if (py < 0 || py >= H || px < 0 || px >= W) continue;
        const long long o = base + (long long)py * W + px;
        const uint32_t q = (uint32_t)idx[o];
        g[i] = gout[o];
        uint32_t qy = __umulhi(q, inv_w);                                   // q / W or one less
        uint32_t qx = q - qy * (uint32_t)W;
        if (qx >= (uint32_t)W) ++qy, qx -= (uint32_t)W;
        const int ly = (int)qy - Y0, lx = (int)qx - X0;                     // place of q in the block
        const int dy = y - ly, dx = x - lx;                                 // place of p in q's window
        if (q < (uint32_t)(H * W) && (uint32_t)ly < (uint32_t)ROWS && (uint32_t)lx < (uint32_t)kBX &&
            (uint32_t)dy < (uint32_t)k && (uint32_t)dx < (uint32_t)k)
            atomicOr(&bits[(dy * RB >> 5) * kQ + ly * kBX + lx], 1u << ((dy * RB & 31) + dx));
    }
    __syncthreads();
    const int tx = threadIdx.x % kBX, ty = threadIdx.x / kBX;
    const int qx = X0 + tx;
    if (qx >= W) return;
    for (int ly = ty; ly < ROWS; ly += THREADS / kBX) {
        if (Y0 + ly >= H) break;
        float acc = 0.0f;
        for (int w = 0; w < words; ++w) {
            const float* p = g + (ly + w * (32 / RB)) * lw + tx;
            uint32_t m = bits[w * kQ + ly * kBX + tx];
            while (m) {
                const int c = __builtin_ctz(m);
                m &= m - 1;
                acc = __fadd_rn(acc, p[c / RB * lw + c % RB]);
            }
        }
        gin[base + (long long)(Y0 + ly) * W + qx] = acc;
    }
}

// Windows beyond 31, and up to 7 with few pixels: every q compares the argmedian
// of its k * k neighbours.
__global__ void __launch_bounds__(kThreads)
mf_grad_gather_kernel(const float* __restrict__ gout, const int32_t* __restrict__ idx,
                      float* __restrict__ gin, int H, int W, int k, int nbx, int nby)
{
    extern __shared__ float g[];
    const int plane = blockIdx.x / (nbx * nby);
    const int b = blockIdx.x - plane * nbx * nby;
    const int by = b / nbx, bx = b - by * nbx;
    const int r = (k - 1) / 2;
    const long long base = (long long)plane * H * W;
    const int X0 = bx * kBX, Y0 = by * kBY;
    const int lw = kBX + 2 * r, lh = kBY + 2 * r;
    int32_t* ix = reinterpret_cast<int32_t*>(g + lw * lh);
    for (int i = threadIdx.x; i < lw * lh; i += kThreads) {
        const int y = i / lw, x = i - y * lw;
        const int py = Y0 - r + y, px = X0 - r + x;
        const bool in = py >= 0 && py < H && px >= 0 && px < W;
        const long long o = base + (long long)py * W + px;
        g[i] = in ? gout[o] : 0.0f;
        ix[i] = in ? idx[o] : -1;   // -1 never equals a pixel index
    }
    __syncthreads();
    const int tx = threadIdx.x % kBX, ty = threadIdx.x / kBX;
    const int qy = Y0 + ty, qx = X0 + tx;
    if (qy >= H || qx >= W) return;
    const int q = qy * W + qx;
    float acc = 0.0f;
    // ascending p = py * W + px: rows top to bottom, columns left to right
    for (int dy = 0; dy < k; ++dy) {
        const int o = (ty + dy) * lw + tx;
        for (int dx = 0; dx < k; ++dx)
            if (ix[o + dx] == q) acc = __fadd_rn(acc, g[o + dx]);
    }
    gin[base + q] = acc;
}

namespace {

template <class F>
hipError_t allow_lds(F fn, size_t lds)
{
    return lds <= 64 * 1024 ? hipSuccess
                            : hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

// launch(p0, np) for planes [p0, p0 + np) at a time: a grid of 2^32 threads or
// more wraps, without an error.
template <class Launch>
hipError_t by_planes(int64_t planes, int64_t plane_blocks, int threads, const Launch& launch)
{
    const int64_t most = ((1LL << 32) - 1) / threads / plane_blocks;
    if (most < 1) return hipErrorInvalidValue;
    for (int64_t p0 = 0; p0 < planes; p0 += most) {
        launch(p0, planes - p0 < most ? planes - p0 : most);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int K, int ROWS>
hipError_t argmedian(const float* src, const float* med, int32_t* idx, int64_t planes, int H, int W, int k,
                     hipStream_t stream)
{
    const int nbx = (W + kBX - 1) / kBX, nby = (H + kBY * ROWS - 1) / (kBY * ROWS);
    const size_t lds = (size_t)(kBX + k - 1) * (kBY * ROWS + k - 1) * 4;
    hipError_t e = allow_lds(mf_argmedian_kernel<K, ROWS>, lds);
    if (e != hipSuccess) return e;
    return by_planes(planes, (int64_t)nbx * nby, kThreads, [&](int64_t p0, int64_t np) {
        const int64_t o = p0 * H * W;
        hipLaunchKernelGGL((mf_argmedian_kernel<K, ROWS>), dim3((unsigned)(np * nbx * nby)), dim3(kThreads), lds, stream,
                           (const uint32_t*)src + o, (const uint32_t*)med + o, idx + o, H, W, k, nbx, nby);
    });
}

template <int RB, int ROWS, int THREADS>
hipError_t grad_bits(const float* gout, const int32_t* idx, float* gin, int64_t planes, int H, int W, int k,
                     hipStream_t stream)
{
    const int nbx = (W + kBX - 1) / kBX, nby = (H + ROWS - 1) / ROWS;
    const int lw = kBX + k - 1, lh = ROWS + k - 1;
    const size_t lds = (size_t)((k * RB + 31) / 32 * kBX * ROWS + lw * lh) * 4;
    const uint32_t inv_w = W == 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (unsigned)W);
    const uint32_t inv_lw = ((1u << 20) + lw - 1) / lw;
    hipError_t e = allow_lds(mf_grad_bits_kernel<RB, ROWS, THREADS>, lds);
    if (e != hipSuccess) return e;
    return by_planes(planes, (int64_t)nbx * nby, THREADS, [&](int64_t p0, int64_t np) {
        const int64_t o = p0 * H * W;
        hipLaunchKernelGGL((mf_grad_bits_kernel<RB, ROWS, THREADS>), dim3((unsigned)(np * nbx * nby)), dim3(THREADS), lds,
                           stream, gout + o, idx + o, gin + o, H, W, k, nbx, nby, inv_w, inv_lw);
    });
}

}  // namespace

hipError_t mf_ag_argmedian_launch(const float* src, const float* med, int32_t* idx, int64_t planes, int H,
                                  int W, int k, hipStream_t stream)
{
    switch (k) {
#define MF_CASE(K) case K: return argmedian<K, 4>(src, med, idx, planes, H, W, k, stream);
    MF_CASE(3) MF_CASE(5) MF_CASE(7) MF_CASE(9) MF_CASE(11) MF_CASE(13) MF_CASE(15)
#undef MF_CASE
    default:
        return H <= 8 || planes * ((W + kBX - 1) / kBX) * ((H + 15) / 16) <= 256
                   ? argmedian<0, 1>(src, med, idx, planes, H, W, k, stream)
                   : argmedian<0, 4>(src, med, idx, planes, H, W, k, stream);
    }
}

hipError_t mf_ag_grad_launch(const float* gout, const int32_t* idx, float* gin, int64_t planes, int H, int W,
                             int k, hipStream_t stream)
{
    const int nbx = (W + kBX - 1) / kBX;
    const bool few = k <= 7 && planes * nbx * ((H + kBY - 1) / kBY) <= 1024;     // work-groups that compare
    if (k <= 7 && !few) return grad_bits<8, 16, 256>(gout, idx, gin, planes, H, W, k, stream);
    if (k <= 15 && !few) return grad_bits<16, 16, 512>(gout, idx, gin, planes, H, W, k, stream);
    if (k <= 31 && !few) return grad_bits<32, 8, 512>(gout, idx, gin, planes, H, W, k, stream);
    const int nby = (H + kBY - 1) / kBY;
    const size_t lds = (size_t)(kBX + k - 1) * (kBY + k - 1) * 8;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)mf_grad_gather_kernel,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return by_planes(planes, (int64_t)nbx * nby, kThreads, [&](int64_t p0, int64_t np) {
        const int64_t o = p0 * H * W;
        hipLaunchKernelGGL(mf_grad_gather_kernel, dim3((unsigned)(np * nbx * nby)), dim3(kThreads), lds, stream, gout + o,
                           idx + o, gin + o, H, W, k, nbx, nby);
    });
}
