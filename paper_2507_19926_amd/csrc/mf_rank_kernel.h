// Ranked sliding-histogram median of 16- and 32-bit planes (kernel templates).
//
// A work-group takes a region of kCols x R outputs. It sorts the region's
// footprint (kCols + KW - 1 columns by R + KH - 1 rows, up to 27 900 values)
// once in LDS, by a stable radix sort of four bits a pass whose counters are
// private to a thread (no ballots: a thread counts its own contiguous run),
// and replaces every value by the 8-bit number of its bucket: bucket b holds
// the S values of ranks b S .. b S + S - 1, whatever their distribution, ties
// included. The histogram of the bucket numbers then slides down the region
// as for 8-bit data (mf_hist_kernel.h) and gives, per output, the bucket of
// the median and the median's place among the bucket's values inside the
// window. That pair is left in the output's own place in dst; last, every
// thread takes outputs in turn and walks the bucket's list of positions in
// rank order, eight at a time, counting those inside the window (two byte
// comparisons by v_lerp_u8 for two positions at once), from the nearer end,
// and stores the value at the position found.
//
// The LDS holds one region per CU: 66 KB of counters, the bucket numbers, and
// the list (2 bytes a value); the sort's buffer lies over all of them.
//
// Bound: one region's latency, two waves to a SIMD. Of a 16-bit region at
// k = 35 the load takes about 12 thousand clocks, the four sort passes 45, the
// bucket numbers 9, the first window 11, the 64 row steps 70 and the walk 32;
// 32-bit data have eight passes over twice the bytes. 4096^2, before (schedule) and now:
// uint16 k = 35 4.33 / 0.66 ms; float32 k = 25 6.3 / 0.84 ms.
#pragma once

#include "mf_hist_kernel.h"

namespace {

typedef __attribute__((address_space(3))) uint16_t lds_u16;

constexpr int kRankThreads = 512;
constexpr int kRankRows = 64;            // output rows of a batched block
constexpr int kRankValues = 27900;       // most values of a footprint: 75 columns' of 64 rows

__device__ __forceinline__ uint32_t rank_key(uint32_t b, bool is_float)
{
    return is_float ? b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u) : b;
}

// V: uint16_t or uint32_t (float32 by its ordered key). KHM: most rows of the
// window.
template <int KW, int KHM, class V, bool TALL = false>
struct Rank {
    typedef Hist<KW, 2> Hs;
    static constexpr int kCols = Hs::kCols;
    static constexpr int FW = kCols + KW - 1;                 // footprint columns
    // Most output rows: 64, or (TALL) as many as the LDS sorts the footprint
    // of, up to 128: a plane of few regions then takes a round of the CUs less
    // (float32 k = 25, 1531 x 2049: 104 rows 187 us, 64 rows 218), the runs of a
    // thread are longer and slower (4096^2: 0.89 ms against 0.84).
    static constexpr int kFit = (kRankValues / FW - (KHM - 1)) / 8 * 8;
    static constexpr int kRows = !TALL ? kRankRows : kFit < 128 ? kFit : 128;
    static_assert(kRows >= kRankRows, "a batched block is a region");
    static constexpr int FHM = kRows + KHM - 1;               // most footprint rows
    static constexpr int FS = Hs::kRow;                       // bytes of a row of bucket numbers
    static constexpr int E = ((FW * FHM + kRankThreads - 1) / kRankThreads) | 1;   // most values of a thread
    static constexpr bool kFull = sizeof(V) == 2 || E <= 45;  // runs that fit the registers (see pass)
    static constexpr int SM = ((FW * FHM + 255) / 256 + 7) / 8 * 8;   // most values of a bucket
    static constexpr uint32_t kIds = kStage;
    static constexpr uint32_t kList = kIds + (FS * FHM + 15) / 16 * 16;
    static constexpr uint32_t kAfter = kList + 2 * 256 * SM;
    static constexpr uint32_t kCnt = E * kRankThreads * 4;    // sort: values, counters [16][threads], totals
    static constexpr uint32_t kTot = kCnt + 16 * kRankThreads * 4;
    static constexpr uint32_t kLds = kAfter > kTot + 64 ? kAfter : kTot + 64;
    static_assert(kLds <= 160 * 1024, "a region fits one CU's LDS");
    static_assert(FW < 255 && FHM < 255, "positions are two bytes");
    static constexpr bool kPacked = sizeof(V) == 2;           // value and position in one word

    static __device__ __forceinline__ uint32_t ld(uint32_t a) { return *(const lds_u32*)(uintptr_t)a; }
    static __device__ __forceinline__ void st(uint32_t a, uint32_t v) { *(lds_u32*)(uintptr_t)a = v; }

    // Inclusive sum over the lanes of a wave.
    static __device__ __forceinline__ uint32_t wave_sum(uint32_t v)
    {
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);    // row_shr 1
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);    // row_shr 2
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);    // row_shr 4
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);    // row_shr 8
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast 15
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast 31
        return v;
    }

    // One stable pass over the four bits from `shift` on of key; pos follows.
    // FULL: eu == E, and the loops over a thread's values have no conditions, so
    // the compiler keeps their LDS accesses in flight together: 4096^2 uint16
    // k = 35 0.67 ms against 0.73, k = 75 1.00 against 1.12, float32 k = 25 0.84
    // against 0.93. Long runs of 32-bit data then spill (k = 75 1.56 against
    // 1.50 ms) and keep the conditions.
    template <bool FULL>
    static __device__ __forceinline__ void pass(uint32_t (&key)[E], uint32_t (&pos)[kPacked ? 1 : E], int shift, int t,
                                                int eu, int n)
    {
        const uint32_t cnt = kCnt + (uint32_t)t * 4;
#pragma unroll
        for (int d = 0; d < 16; ++d) st(cnt + d * (kRankThreads * 4), 0);
        uint32_t r[E];
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (FULL || j < eu) r[j] = __hip_atomic_fetch_add((lds_u32*)(uintptr_t)(cnt + ((key[j] >> shift) & 15u) * (kRankThreads * 4)), 1u,
                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        // exclusive sums, digit by digit and thread by thread: a wave takes
        // two digits, a lane eight threads' counters
        const int lane = t & 63, wave = t >> 6;
        uint32_t v[2][8], run[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t a = kCnt + (uint32_t)((wave * 2 + q) * kRankThreads + lane * 8) * 4;
            const u32x4 x = *(const lds_u32x4*)(uintptr_t)a, y = *(const lds_u32x4*)(uintptr_t)(a + 16);
            v[q][0] = x.x, v[q][1] = x.y, v[q][2] = x.z, v[q][3] = x.w;
            v[q][4] = y.x, v[q][5] = y.y, v[q][6] = y.z, v[q][7] = y.w;
            uint32_t s = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) s += v[q][i];
            const uint32_t inc = wave_sum(s);
            run[q] = inc - s;
            if (lane == 63) st(kTot + (uint32_t)(wave * 2 + q) * 4, inc);
        }
        __syncthreads();
        // nothing to do where all values have the same four bits (the fillers,
        // last already, have bits 15)
        const uint32_t tot = ld(kTot + (lane & 15) * 4);
        if (__any(tot >= (uint32_t)n + ((lane & 15) == 15 ? (uint32_t)(kRankThreads * eu - n) : 0u))) {
            __syncthreads();
            return;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            uint32_t b = run[q];
            for (int d = 0; d < wave * 2 + q; ++d) b += (uint32_t)__builtin_amdgcn_readlane((int)tot, d);
            const uint32_t a = kCnt + (uint32_t)((wave * 2 + q) * kRankThreads + lane * 8) * 4;
            uint32_t o[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = b, b += v[q][i];
            *(lds_u32x4*)(uintptr_t)a = u32x4{o[0], o[1], o[2], o[3]};
            *(lds_u32x4*)(uintptr_t)(a + 16) = u32x4{o[4], o[5], o[6], o[7]};
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < E; ++j) if (FULL || j < eu) {
            r[j] = (r[j] + ld(cnt + ((key[j] >> shift) & 15u) * (kRankThreads * 4))) * 4;
            st(r[j], key[j]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < E; ++j) if (FULL || j < eu) key[j] = ld((uint32_t)(t * eu + j) * 4);
        __syncthreads();
        if constexpr (!kPacked) {
#pragma unroll
            for (int j = 0; j < E; ++j) if (FULL || j < eu) st(r[j], pos[j]);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < E; ++j) if (FULL || j < eu) pos[j] = ld((uint32_t)(t * eu + j) * 4);
            __syncthreads();
        }
    }

    // Place in its group of eight list entries of the q-th of them in rank
    // order: the flags of a group then come out in rank order (see walk()).
    static __device__ __forceinline__ uint32_t place(uint32_t q) { return q < 4 ? 2 * q : 2 * q - 7; }

    static __device__ __forceinline__ void region(const unsigned char* __restrict__ src, unsigned char* dst, int H, int W,
                                                  long long pitch, int x0, int y0, int y1, int kh, bool is_float)
    {
        const int t = (int)threadIdx.x, lane = t & 63;
        const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
        const int rows = y1 - y0, fh = rows + kh - 1, n = FW * fh;
        const int rx = KW / 2, ry = kh / 2;
        const int S = ((n + 255) / 256 + 7) / 8 * 8;
        auto at = [&](int fy, int fx) {
            return src + (long long)min(max(y0 - ry + fy, 0), H - 1) * pitch +
                   (long long)min(max(x0 - rx + fx, 0), W - 1) * (int)sizeof(V);
        };
        {
            // footprint into the buffer, rows dealt to the waves, four in flight
            {
                constexpr int NX = (FW + 63) / 64;
                uint32_t gx[NX];
#pragma unroll
                for (int i = 0; i < NX; ++i)
                    gx[i] = (uint32_t)min(max(x0 - rx + lane + 64 * i, 0), W - 1) * (uint32_t)sizeof(V);
                for (int f0 = wave; f0 < fh; f0 += 32) {
                    uint32_t v[4][NX];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const unsigned char* rowp =
                            src + (long long)min(max(y0 - ry + min(f0 + 8 * q, fh - 1), 0), H - 1) * pitch;
#pragma unroll
                        for (int i = 0; i < NX; ++i) v[q][i] = *(const V*)(rowp + gx[i]);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int i = 0; i < NX; ++i)
                            if (f0 + 8 * q < fh && lane + 64 * i < FW)
                                st((uint32_t)((f0 + 8 * q) * FW + lane + 64 * i) * 4, rank_key(v[q][i], is_float));
                }
            }
            __syncthreads();
            // row-major runs, one to a thread, of an odd number of values (a
            // run then starts in another LDS bank than its neighbours'); the
            // fillers come last and stay last (stable sort)
            const int need = ((n + kRankThreads - 1) / kRankThreads) | 1;
            const bool full = kFull && need * 8 >= E * 7;
            const int eu = full ? E : need;
            uint32_t key[E], pos[kPacked ? 1 : E];
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const int i = t * eu + j, fy = i / FW, fx = i - fy * FW;
                const bool real = j < eu && i < n;
                const uint32_t p = real ? (uint32_t)(fy << 8 | fx) : 0xffffu;
                const uint32_t v = ld((uint32_t)i * 4);       // in the buffer, whatever i
                const uint32_t k = real ? v : 0xffffffffu;
                if constexpr (kPacked) key[j] = k << 16 | p;
                else key[j] = k, pos[j] = p;
            }
            __syncthreads();
            for (int s = kPacked ? 16 : 0; s < 32; s += 4) {
                if (full) pass<kFull>(key, pos, s, t, eu, n);
                else pass<false>(key, pos, s, t, eu, n);
            }
            // bucket numbers and list; i / S = i * inv >> 22 for i < 2^22 / S
            static_assert((long long)E * kRankThreads * SM < (1 << 22) && SM <= 255, "i / S by one product");
            const uint32_t inv = (uint32_t)(((1 << 22) + S - 1) / S);
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const uint32_t i = j < eu ? (uint32_t)(t * eu + j) : 0xffffffffu;
                const uint32_t p = kPacked ? key[j] & 0xffffu : pos[kPacked ? 0 : j];
                if (i < (uint32_t)n)
                    *(lds_u8*)(uintptr_t)(kIds + (p >> 8) * FS + (p & 255u)) = (uint8_t)(__umul24(i, inv) >> 22);
                if (i < 256u * (uint32_t)S)
                    *(lds_u16*)(uintptr_t)(kList + 2 * ((i & ~7u) + place(i & 7u))) = (uint16_t)p;
            }
            for (uint32_t i = (uint32_t)(eu * kRankThreads + t); i < 256u * (uint32_t)S; i += kRankThreads)
                *(lds_u16*)(uintptr_t)(kList + 2 * i) = 0xffffu;
            for (uint32_t i = (uint32_t)t * 16; i < kStage; i += kRankThreads * 16)
                *(lds_u32x4*)(uintptr_t)i = u32x4{0, 0, 0, 0};
        }
        __syncthreads();

        // slide: waves 0 and 1 search, 2 and 3 slide, the others join for the
        // first window
        const uint32_t g4 = 4u * (uint32_t)(lane & 31);
        const int sub = lane >> 5;
        if (wave < 2) {
            const int w = 2 * wave + sub;
            const int ox = (int)g4 + w;
            uint32_t nge = 0, m = 128, nm = ~(m * 0x01010101u);
            for (int q = 0; q < kh; ++q) {
                uint32_t d[Hs::ND];
                Hs::read_row(d, kIds + q * FS + g4);
                nge = Hs::count_ge(d, nm, w, nge);
            }
            const int all = KW * kh;
            int e = (all - 1) / 2 - (all - (int)nge);
            uint32_t am = (m << 8) + g4 + kPad;
            __syncthreads();
            const bool inside = x0 + ox < W;
            unsigned char* out = dst + (long long)y0 * pitch + (long long)(x0 + ox) * (int)sizeof(V);
            for (int y = 0; y < rows; ++y) {
                int more = 0;
                int back = Hs::find(am, e, w, more);
                __syncthreads();
                asm volatile("" : "+v"(am), "+v"(e), "+v"(back));
                m = ((am - kPad) >> 8) & 255u;
                const uint32_t code = m | (uint32_t)min(e, back) << 8 | (back < e ? 0x8000u : 0u);
                if (inside) *(V*)out = (V)code;
                out += pitch;
                if (y + 1 < rows) {
                    uint32_t din[Hs::ND], dout[Hs::ND];
                    Hs::read_row(din, kIds + (uint32_t)(y + kh) * FS + g4);
                    Hs::read_row(dout, kIds + (uint32_t)y * FS + g4);
                    nm = ~__builtin_amdgcn_perm(m, m, 0u);
                    e = (int)(Hs::count_ge(din, nm, w, (uint32_t)e) - Hs::count_ge(dout, nm, w, 0));
                }
                asm volatile("" : "+v"(e));
                __syncthreads();
            }
        } else {
            for (int q = (wave - 2) * 2 + sub; q < kh; q += 12) {
                uint32_t d[1][Hs::ND];
                Hs::read_row(d[0], kIds + q * FS + g4);
                Hs::template update<0, Hs::NG, false, false>(d, g4, 1);
            }
            __syncthreads();
            if (wave < 4) {
                const int one = sub ? -1 : 1;
                for (int y = 0; y < rows; ++y) {
                    uint32_t d[1][Hs::ND];
                    // past the last step the counters are not read any more
                    Hs::read_row(d[0], kIds + (uint32_t)(sub || y + 1 == rows ? y : y + kh) * FS + g4);
                    if (wave == 3) Hs::template update<Hs::CH, Hs::NG, true, false>(d, g4, one);
                    else Hs::template update<0, Hs::CH, true, false>(d, g4, one);
                    __syncthreads();
                }
            } else {
                for (int y = 0; y < rows; ++y) {
                    __syncthreads();
                    __syncthreads();
                }
            }
        }

        // walk: every thread takes a column and every fourth row, four
        // outputs at a time: a list read waits for its bank conflicts, not
        // for its instructions
        constexpr int kStepRows = kRankThreads / kCols;
        const int ox = t & (kCols - 1), oy0 = t / kCols;
        const bool inx = x0 + ox < W;
        unsigned char* const col = dst + (long long)y0 * pitch + (long long)(x0 + ox) * (int)sizeof(V);
        for (int yb = oy0; yb < rows; yb += 4 * kStepRows) {
            // a thread reads the codes of its own outputs only: the others'
            // may hold their medians already
            Walk k[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int oy = yb + q * kStepRows;
                const bool own = inx && oy < rows;
                k[q] = begin(own ? (uint32_t)*(const V*)(col + (long long)oy * pitch) : 0u, ox, oy, kh, S);
                k[q].e = own ? k[q].e : -1;
            }
            for (int g = 0; g < S / 8; ++g) {
                u32x4 x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = fetch(k[q]);
                bool more = false;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    count(k[q], x[q]);
                    more |= k[q].e >= k[q].c;
                }
                if (!__any(more)) break;
            }
            uint32_t val[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t p = end(k[q]);
                val[q] = *(const V*)at((int)(p >> 8), (int)(p & 255u));
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (inx && yb + q * kStepRows < rows) *(V*)(col + (long long)(yb + q * kStepRows) * pitch) = (V)val[q];
        }
    }

    // A walk through a bucket's list.
    struct Walk {
        uint32_t nlo, nhi, a, step, f;
        int e, c;
        bool back;
    };
    // code: bucket, number of entries inside the window before the median's,
    // bit 15: from the bucket's end; window at (ox, oy) of the footprint.
    static __device__ __forceinline__ Walk begin(uint32_t code, int ox, int oy, int kh, int S)
    {
        Walk k;
        const uint32_t lo = (uint32_t)(oy << 8 | ox) * 0x00010001u;
        k.nlo = ~lo;
        k.nhi = ~(lo + (uint32_t)(kh << 8 | KW) * 0x00010001u);
        k.back = (code & 0x8000u) != 0;
        k.e = (int)((code >> 8) & 127u);
        k.step = k.back ? 0u - 16u : 16u;
        k.a = kList + __umul24(code & 255u, (uint32_t)(2 * S)) + (k.back ? (uint32_t)(2 * S) - 16u : 0u) - k.step;
        k.c = 0;
        k.f = 0;
        return k;
    }
    // The next eight entries, or the last eight again once the median's is
    // among them; both are in the list.
    static __device__ __forceinline__ u32x4 fetch(Walk& k)
    {
        const bool on = k.e >= k.c;
        k.e -= on ? k.c : 0;
        k.a += on ? k.step : 0u;
        return *(const lds_u32x4*)(uintptr_t)k.a;
    }
    static __device__ __forceinline__ void count(Walk& k, const u32x4& x)
    {
        constexpr uint32_t kTop = 0x80008000u;
        uint32_t f = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t wd = i == 0 ? x.x : i == 1 ? x.y : i == 2 ? x.z : x.w;
            // top bits: byte >= first coordinate, and not >= the one past the last
            uint32_t in = __builtin_amdgcn_lerp(wd, k.nlo, 0x01010101u) & ~__builtin_amdgcn_lerp(wd, k.nhi, 0x01010101u);
            in &= in << 8;
            f = (f >> 1) | (in & kTop);
        }
        k.f = f;
        k.c = __builtin_popcount(f);
    }
    // Position of the entry: the flags of a group's entries in rank order are
    // bits 12..15 and 28..31.
    static __device__ __forceinline__ uint32_t end(const Walk& k)
    {
        int r = k.back ? k.c - 1 - k.e : k.e;
        const int low = __builtin_popcount(k.f & 0xffffu);
        uint32_t nib = r < low ? (k.f >> 12) & 15u : k.f >> 28;
        const uint32_t half = r < low ? 0u : 2u;
        r = r < low ? r : r - low;
#pragma unroll
        for (int i = 0; i < 3; ++i) nib = i < r ? nib & (nib - 1) : nib;
        return *(const lds_u16*)(uintptr_t)(k.a + (uint32_t)__builtin_ctz(nib | 16u) * 4 + half);
    }
};

template <int KW, int KHM, class V, bool TALL>
__global__ void __launch_bounds__(kRankThreads)
mf_rank_kernel(const unsigned char* __restrict__ src, unsigned char* dst, int H, int W, long long pitch,
               long long plane_stride, int ncol, int R, int kh, int is_float, int b0)
{
    typedef Rank<KW, KHM, V, TALL> Rk;
    const int b = b0 + (int)blockIdx.x, cb = b % ncol, s = b / ncol;
    const long long po = (long long)blockIdx.y * plane_stride;   // plane = blockIdx.y
    Rk::region(src + po, dst + po, H, W, pitch, cb * Rk::kCols, s * R, min((s + 1) * R, H), kh, is_float != 0);
}

// Square windows of a job table (MfJob), kRankRows output rows to a block.
template <int KW, int KHM, class V>
__global__ void __launch_bounds__(kRankThreads)
mf_rank_kernel_batched(const MfJob* __restrict__ jobs, int njobs, int nblocks)
{
    typedef Rank<KW, KHM, V> Rk;
    for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
        int lo = 0, hi = njobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (jobs[mid].block_begin <= b) lo = mid;
            else hi = mid - 1;
        }
        const MfJob j = jobs[lo];
        const int lb = b - j.block_begin;
        const int y0 = lb / j.nbx * kRankRows;
        Rk::region(j.src, j.dst, j.H, j.W, j.pitch, lb % j.nbx * Rk::kCols, y0, min(y0 + kRankRows, j.H), KW,
                   j.dtype == MF_F32);
        __syncthreads();   // the next block reuses the LDS
    }
}

template <int KW, int KHM, class V, bool BATCHED>
HistKernelInfo rank_kernel()
{
    typedef Rank<KW, KHM, V> Rk;
    const void* b = nullptr;
    if constexpr (BATCHED) b = (const void*)mf_rank_kernel_batched<KW, KHM, V>;
    HistKernelInfo k = {(const void*)mf_rank_kernel<KW, KHM, V, false>, b, kRankThreads, Rk::kCols, kRankRows, Rk::kLds,
                        Rk::kRows};
    if constexpr (sizeof(V) == 4 && Rk::kFit > kRankRows) {
        typedef Rank<KW, KHM, V, true> Tall;
        k.tall = (const void*)mf_rank_kernel<KW, KHM, V, true>;
        k.tall_lds = Tall::kLds;
        k.max_rows = Tall::kRows;
    }
    return k;
}

}  // namespace
