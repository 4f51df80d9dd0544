// Sliding-histogram median of 8-bit planes (kernel templates; mf_hist.hip and
// its parts instantiate them).
//
// A work-group walks down a strip of kCols output columns and keeps, in LDS,
// the histogram of every column's window while the window slides by one row.
// Neighbouring columns share their windows' inner columns, so four adjacent
// columns form a group with one set of 256 counter words: the count of the
// KW - 3 columns that all four windows hold, and the counts of the three
// columns left (L0 L1 L2) and right (R0 R1 R2) of them; window w of the group
// is the shared count and three consecutive ones of L0 L1 L2 R0 R1 R2, summed
// by one or two dot products of the counter word. A row step costs
// 2 (KW + 3) LDS atomics per group of four pixels whatever the data, against
// the hundreds of merge outputs or min/max per pixel of the schedules and
// networks, and no work grows with KW * KH.
//
// Counter words: P = 1 holds all seven counts in 32 bits (8 shared, six of 4;
// windows of up to 15 rows and 255 shared values), 64 groups to a
// work-group; P = 2 in 64 bits (16 shared, six of 8), 32 groups. Either way
// 64 KB of counters and 4 KB for 16 bins each, two work-groups per CU. A field may overflow between an
// addition and the removal that follows it: words are added modulo 2^32, so
// they are exact when read. Bin v of group g lies at 256 v + 128 p + 4 g:
// the address of a pixel's counter is one v_perm_b32 (pixel byte above the
// group's byte), and no two groups of a wave share an LDS bank.
//
// Half of the waves search, half slide the histogram, in turn (two barriers
// a row). A search wave starts at the last median's bin: it knows how many
// window values lie below that bin (the rows that came and went are counted
// against it, four bytes at a time, by v_lerp_u8's carry) and walks up or
// down from it, four bins and then eight at a time. Where the walks are long
// (two levels, noise), counters of 16 bins are kept too and searched instead
// (see rows()). A slide wave holds the addresses of its counters ready while
// the others search.
//
// Bound: the row step's latency (a barrier, the dependent search, a barrier,
// the atomics), overlapped between the two work-groups of a CU; from about
// k = 50 on the LDS atomics (4.0 clocks of the CU for each wave's, 14.6 for one
// wave alone). Per 30 MP RGB frame (smooth image), before (network, schedule)
// and now: k = 17 1.41 / 0.56 ms, k = 25 10.4 / 0.65, k = 75 40.2 / 1.39.
#pragma once

#include <type_traits>

#include "mf_hist.h"

#define MF_HOST_DEVICE __host__ __device__
#include "mf_hist_role.h"

namespace {

typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) u32x4a4 lds_u32x4a4;

constexpr int kT = 4;                 // output columns of a group
// Room before the counters and after them: a lane whose median is found reads
// on with the lanes that still walk, eight bins from its own each time, so
// up to seven bins past either end. What it reads there is not used.
constexpr uint32_t kPad = 2048;
constexpr uint32_t kCounters = 65536;
constexpr uint32_t kStage = kPad + kCounters + kPad;

// Counter words of a group: P = 1: one, 64 groups to a work-group, bin v of
// group g at 256 v + 4 g; P = 2: two, 32 groups, word p at 256 v + 128 p + 4 g.
template <int KW, int P, int Z = 1>
struct Hist {
    static constexpr int kGroups = 64 / P;
    static constexpr int kCols = kGroups * kT;          // output columns of a work-group
    static constexpr int kWaves = kT / P;               // search waves, and update waves
    static constexpr int kThreads = 2 * 64 * kWaves;
    static constexpr int NG = KW + kT - 1;              // columns of a group's windows
    static constexpr int ND = (NG + 3) / 4;             // dwords of them
    static constexpr int NB = kT * (kGroups - 1) + 4 * ND;   // bytes of a staged row
    static constexpr int kRow = (NB + 15) / 16 * 16;
    static constexpr int NL = (kRow + 63) / 64;         // byte loads of a whole row
    static constexpr int NF = P == 1 ? (kRow + 127) / 128 : NL;   // of a wave's part of a row
    static constexpr int CH = (ND + 1) / 2 * 4;         // columns of the first half of a row
    // staged rows: [2 steps][in, out][Z slices]; the first window takes them four
    // at a time. They hold whole loads, so that a store needs no condition (30 MP
    // k = 17, smooth 208 us with conditions, 198 without)
    static constexpr int kStaged = P == 1 ? 128 * NF : 64 * NL;
    static constexpr uint32_t kRowsEnd = kStage + 4 * Z * kStaged;
    // planes: counters of 16 bins each, as the bins' own at 256 v + 128 p + 4 g;
    // a word in which a search wave asks for them, and one in which each says
    // whether to go on with them
    static constexpr bool kCoarse = Z == 1;
    static constexpr uint32_t kAsk = kRowsEnd + 16 * 256;
    static constexpr uint32_t kKeep = kAsk + 16;
    static constexpr uint32_t kLds = kCoarse ? kKeep + 16 : kRowsEnd;
    static_assert(kLds <= 80 * 1024, "two work-groups to a CU");
    static constexpr int kFar = 4;       // probes of eight bins a row from which the counters of 16 bins pay
    static constexpr int kFarRows = 16;  // rows for which they are kept at least

    // Column i of a group adds 1 << shift(i) to word(i).
    static constexpr int word(int i) { return P == 2 && (i == 2 || i >= KW); }
    static constexpr int shift(int i)
    {
        if (i >= 3 && i < KW) return 0;
        const int f = i < 3 ? i : 3 + i - KW;           // L0 L1 L2 R0 R1 R2
        return P == 1 ? 8 + 4 * f : f < 2 ? 16 + 8 * f : 8 * (f - 2);
    }

    // flags of the group's bytes that lie in the window of output column w
    static __device__ __forceinline__ uint32_t keep(int j, int w)
    {
        uint32_t m = 0x80808080u;
        if (j == 0) m <<= 8 * w;
        if (4 * j + 4 > KW) {                           // bytes w + KW and on are outside
            const int n = w + KW - 4 * j;               // bytes of this dword inside
            m = n >= 4 ? m : n <= 0 ? 0u : m & (0xffffffffu >> (32 - 8 * n));
        }
        return m;
    }
    // acc + number of the window's bytes >= m; nm = ~m in every byte. v_lerp
    // gives (x + ~m + 1) >> 1 per byte, whose top bit is the carry: x >= m.
    static __device__ __forceinline__ uint32_t count_ge(const uint32_t (&d)[ND], uint32_t nm, int w, uint32_t acc)
    {
#pragma unroll
        for (int j = 0; j < ND; ++j)
            acc = __builtin_popcount(__builtin_amdgcn_lerp(d[j], nm, 0x01010101u) & keep(j, w)) + acc;
        return acc;
    }
    // window counts of output column w in N bins from address a on, st apart
    template <int N>
    static __device__ __forceinline__ void bins(int (&v)[N], uint32_t a, int st, int w)
    {
        uint32_t d[N][P];
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int q = 0; q < P; ++q) d[i][q] = *(const lds_u32*)(uintptr_t)(a + (uint32_t)(i * st) + 128u * q);
        // all reads on their way before the first is waited for
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (P == 1) {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = (int)__builtin_amdgcn_udot8(d[i][0], 0x11100u << (4 * w), d[i][0] & 255u, false);
        } else {
            // three of L0 L1 (word 0, bytes 2 and 3), L2 R0 R1 R2 (word 1)
            const uint32_t mA = 0x01010000u << (8 * w);
            const uint32_t mB = w == 3 ? 0x01010100u : 0x01010101u >> (8 * (3 - w));
#pragma unroll
            for (int i = 0; i < N; ++i)
                v[i] = (int)__builtin_amdgcn_udot4(d[i][P - 1], mB, __builtin_amdgcn_udot4(d[i][0], mA, d[i][0] & 0xffffu, false),
                                                   false);
        }
    }
    static __device__ __forceinline__ void read_row(uint32_t (&d)[ND], uint32_t loc)
    {
#pragma unroll
        for (int j = 0; j + 4 <= ND; j += 4) {
            const u32x4a4 v = *(const lds_u32x4a4*)(uintptr_t)(loc + 4 * j);
            d[j] = v.x, d[j + 1] = v.y, d[j + 2] = v.z, d[j + 3] = v.w;
        }
#pragma unroll
        for (int j = ND & ~3; j < ND; ++j) d[j] = *(const lds_u32*)(uintptr_t)(loc + 4 * j);
    }

    // Adds one (or removes: one = -1) for the bytes of columns [C0, C1) of
    // the group in R rows, with COARSE to the counters of 16 bins too. With
    // SYNC, the addresses are formed before a work-group barrier and the
    // counters change after it.
    template <int C0, int C1, bool SYNC, bool COARSE, int R>
    static __device__ __forceinline__ void update(const uint32_t (&d)[R][ND], uint32_t g4, int one)
    {
        uint32_t a[R][C1 - C0], c[C1 - C0];
        auto at = [&](uint32_t q, int i) {
            return __builtin_amdgcn_perm(q, word(i) ? g4 | 128u : g4, 0x0c0c0000u | ((4u + (i & 3)) << 8));
        };
        auto add = [&](uint32_t loc, int i) {
            __hip_atomic_fetch_add((lds_u32*)(uintptr_t)loc, (uint32_t)one << shift(i), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        };
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = C0; i < C1; ++i) a[r][i - C0] = at(d[r][i / 4], i);
        if constexpr (COARSE) {
#pragma unroll
            for (int i = C0; i < C1; ++i) c[i - C0] = at((d[0][i / 4] >> 4) & 0x0f0f0f0fu, i);
        }
        if constexpr (COARSE) {
            // not sunk past the barrier
#pragma unroll
            for (int i = C0; i < C1; ++i) asm volatile("" : "+v"(a[0][i - C0]), "+v"(c[i - C0]));
        }
        if (SYNC) __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = C0; i < C1; ++i) add(a[r][i - C0] + kPad, i);
        if constexpr (COARSE) {
#pragma unroll
            for (int i = C0; i < C1; ++i) add(c[i - C0] + kRowsEnd, i);
        }
    }

    // The row steps of [y0, y1) by twos, for all waves alike. near(y) does steps
    // y and y + 1 and returns whether a search wave has asked for the counters
    // of 16 bins; far(y) does them with those; keep(n) leaves a search wave's
    // word on the last n rows.
    //
    // The walk from one row's median to the next takes a probe for eight bins,
    // up to 31 of 490 clocks on images of two levels, where a network's time
    // does not depend on the data. With the counters of 16 bins a search reads
    // 16 counters twice, whatever the data, but every row's updates and searches
    // are longer, so they are kept only while the walks are long. A plane of
    // 4480 x 6720 of two levels, us by walks alone / now (network): k = 13 1840 /
    // 277 (325), k = 15 1866 / 294 (399), k = 17 2740 / 471 (495), k = 21 2756 / 494
    // (1226). The question itself costs a smooth image 2 to 5 % of its time (k = 21
    // 12 %, 193 / 217); asking every 16 rows, by a barrier of its own, cost as
    // much, since the rows on their way to the registers are waited for there.
    //
    // The counters of 16 bins are summed from the bins' own where they begin: a
    // field of a counter word over all 256 bins holds no more than a column's or
    // the shared columns' values, so words of any bins add up without a carry.
    //
    // The word kAsk is written before the first barrier of step y + 1 and read by
    // all waves before the second, and cleared after one more: all waves go the
    // same way.
    template <class Near, class Far, class Keep>
    static __device__ __forceinline__ void rows(int y0, int y1, int wave, int lane, const Near& near, const Far& far,
                                                const Keep& keep)
    {
        for (int y = y0;;) {
            bool ask;
            do {
                ask = near(y);
                y += 2;
            } while (y < y1 && !ask);
            if (!kCoarse || y >= y1) return;
            for (int c = wave; c < 16; c += 2 * kWaves) {
                const uint32_t a = kPad + (uint32_t)(c * 16 * 256 + 4 * lane);
                uint32_t sum = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) sum += *(const lds_u32*)(uintptr_t)(a + 256 * i);
                *(lds_u32*)(uintptr_t)(kRowsEnd + (uint32_t)(c * 256 + 4 * lane)) = sum;
            }
            __syncthreads();
            if (wave == 0 && lane == 0) *(lds_u32*)(uintptr_t)kAsk = 0;
            u32x4 on;
            do {
                const int begin = y, end = min(y + kFarRows, y1);
                for (; y < end; y += 2) far(y);
                if (y >= y1) return;
                keep(y - begin);
                __syncthreads();
                on = *(const lds_u32x4*)(uintptr_t)kKeep;
            } while (__builtin_amdgcn_readfirstlane((int)(on.x | on.y | on.z | on.w)) != 0);
        }
    }

    // The wave's number among search (0 .. kWaves - 1) and slide waves. With
    // four waves to a work-group (P = 2) and two work-groups to a CU, each
    // SIMD has two waves; up to about 40 counter updates a row a search wave
    // has more to do than a slide wave, so the work-group that holds the
    // lower half of the CU's LDS searches on SIMDs 0 and 1, the other one on 2
    // and 3, and no two searches share a SIMD. Clocks a row step, smooth image
    // (uniform noise): k = 7 825 (3410) with roles by wave number, 790 (2690)
    // now; k = 17 1005 (1620), 940 (1390); k = 35 1430 (1560), 1270 (1390);
    // k = 65 2010, 1970; k = 75 2270, 2370, so the widest windows keep the wave
    // numbers, and the boxes beyond 9 (k = 15 1.71 ms, 1.75).
    // Only the speed rests on what the registers say: every wave takes its role
    // from the same four published words, whose roles always differ.
    static constexpr bool kBySimd = P == 2 && (Z == 1 ? KW <= 67 : Z <= 9);
    static __device__ __forceinline__ int role()
    {
        int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        if constexpr (kBySimd) {
            constexpr int kSimd = 4 | 4 << 6 | 1 << 11;          // HW_ID bits 4..5
            constexpr int kLdsBase = 6 | 0 << 6 | 11 << 11;      // LDS_ALLOC bits 0..11
            const uint32_t word = hist_role_word(__builtin_amdgcn_s_getreg(kSimd), __builtin_amdgcn_s_getreg(kLdsBase));
            if (__lane_id() == 0) *(lds_u32*)(uintptr_t)(kStage + 4 * wave) = word;
            __syncthreads();
            uint32_t words[4];
            for (int i = 0; i < 4; ++i)
                words[i] = __builtin_amdgcn_readfirstlane((int)*(const lds_u32*)(uintptr_t)(kStage + 4 * i));
            wave = __builtin_amdgcn_readfirstlane(hist_role(words, wave));
            __syncthreads();
        }
        return wave;
    }

    // Rows [y0, y1) of the kCols columns from x0 on. For boxes (Z > 1) of
    // slice z: src is the volume, slices `slice` bytes apart, D of them.
    static __device__ __forceinline__ void strip(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst,
                                                 int H, int W, long long pitch, int x0, int y0, int y1, int kh,
                                                 int D = 1, long long slice = 0, int z = 0)
    {
        const int lane = (int)__lane_id();
        const int wave = role();
        for (uint32_t i = threadIdx.x * 16; i < kStage; i += kThreads * 16)
            *(lds_u32x4*)(uintptr_t)i = u32x4{0, 0, 0, 0};
        if (kCoarse && threadIdx.x == 0) {
            *(lds_u32*)(uintptr_t)kAsk = 0;
            *(lds_u32x4*)(uintptr_t)kKeep = u32x4{0, 0, 0, 0};
        }
        // row y of the q-th slice of the box
        auto row = [&](int y, int q) {
            const unsigned char* p = src + (long long)min(max(y, 0), H - 1) * pitch;
            return Z == 1 ? p : p + (long long)min(max(z - Z / 2 + q, 0), D - 1) * slice;
        };
        if (wave < kWaves) search(row, dst, W, pitch, x0, y0, y1, kh, wave, lane);
        else slide(row, W, x0, y0, y1, kh, wave - kWaves, lane);
    }

    // N counters from address a on, st apart, against the n values of the window
    // that are to be passed: the number of counters passed (N: all), n becomes
    // the rest and hi the complement of the values of the first counter not
    // passed that rank above.
    template <int N>
    static __device__ __forceinline__ int probe(uint32_t a, int st, int w, int& n, uint32_t& hi)
    {
        int v[N];
        bins<N>(v, a, st, w);
        uint32_t lo = (uint32_t)n;
        hi = 0;
        int c = N, r = n;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            r -= v[i];
            lo = min(lo, (uint32_t)r);
            hi = max(hi, (uint32_t)r);
            c += r >> 31;
        }
        n = (int)lo;
        return c;
    }

    // Next median of a lane: e = rank of the median - number of window values
    // below bin m, am = address of bin m; both move to the median's bin.
    // Returns the number of window values of that bin that rank above; more
    // counts the probes after the first.
    static __device__ __forceinline__ int find(uint32_t& am, int& e, int w, int& more)
    {
        const int sg = e >> 31;
        const int st = sg ? -256 : 256;
        uint32_t a = am + (uint32_t)(sg & -256);
        int n = e ^ sg;
        uint32_t hi;
        int c = probe<4>(a, st, w, n, hi);
        a += (uint32_t)(st * c);
        if (__any(c == 4))
            do {
                c = probe<8>(a, st, w, n, hi);
                a += (uint32_t)(st * c);
                ++more;
            } while (__any(c == 8));
        am = a;
        e = sg ? (int)~hi : n;
        return sg ? n : (int)~hi;
    }

    // The same by the counters of 16 bins: rank = rank of the median in the
    // window. more: about what find() would have probed, by two distances.
    static __device__ __forceinline__ void find_coarse(uint32_t& am, int& e, int w, uint32_t g4, int rank, int& more)
    {
        uint32_t hi, a = kRowsEnd + g4;
        int n = rank;
        asm("" : "+v"(a));     // one base for all reads
        a = kPad + g4 + ((uint32_t)probe<16>(a, 256, w, n, hi) << 12);
        a += (uint32_t)probe<16>(a, 256, w, n, hi) << 8;
        const int far = abs((int)(a - am)) >> 8;
        more += (__any(far > 28) ? 4 : 0) + (__any(far > 124) ? 12 : 0);
        am = a;
        e = n;
    }

    template <class Row>
    static __device__ __forceinline__ void search(const Row& row, unsigned char* __restrict__ dst, int W, long long pitch,
                                                  int x0, int y0, int y1, int kh, int wave, int lane)
    {
        const int ry = kh / 2;
        const int w = P == 1 ? wave : 2 * wave + (lane >> 5);
        const uint32_t vo = (uint32_t)(x0 + 4 * (lane & (kGroups - 1)) + w);
        // lanes outside the image search with the last group inside: the windows
        // of the columns they stand for are the last column's values alone,
        // whose medians can jump where the image's do not
        const uint32_t g4 = 4u * (uint32_t)(min(lane & (kGroups - 1), max(W - 1 - x0 - w, 0) >> 2) & (kGroups - 1));
        const bool inside = (int)vo < W;
        uint32_t m;
        {
            const uint32_t xo = (uint32_t)min(x0 + (int)g4 + w, W - 1);
            const uint32_t a = row(y0 - ry, Z / 2)[xo], b = row(y0, Z / 2)[xo], c = row(y0 + ry, Z / 2)[xo];
            m = max(min(a, b), min(max(a, b), c));
        }
        uint32_t nge = 0, nm = ~(m * 0x01010101u);
        for (int j = 0; j < kh * Z; j += 4) {
            __syncthreads();
            for (int q = 0; q < 4 && j + q < kh * Z; ++q) {
                uint32_t d[ND];
                read_row(d, kStage + q * kStaged + g4);
                nge = count_ge(d, nm, w, nge);
            }
            __syncthreads();
        }
        const int all = KW * kh * Z;
        int e = (all - 1) / 2 - (all - (int)nge);
        uint32_t am = (m << 8) + g4 + kPad;
        __syncthreads();
        unsigned char* out = dst + (long long)y0 * pitch;
        int more = -32;      // the first walk starts from a guess and says nothing of the next
        uint32_t ask = 0;
        int asked = 0;
        auto step = [&](auto coarse, int y, int par) {
            if constexpr (decltype(coarse)::value) find_coarse(am, e, w, g4, (all - 1) / 2, more);
            else find(am, e, w, more);
            if (kCoarse && !decltype(coarse)::value && par == 1)
                if (more >= 4 * kFar) *(lds_u32*)(uintptr_t)kAsk = 1;
            __syncthreads();
            // the counters change from here to the next barrier; the median
            // found and its rank in the next window do not depend on them
            asm volatile("" : "+v"(am), "+v"(e));
            if (kCoarse && !decltype(coarse)::value && par == 1) ask = *(const lds_u32*)(uintptr_t)kAsk;
            m = ((am - kPad) >> 8) & 255u;
            if (inside && y < y1) out[vo] = (unsigned char)m;
            out += pitch;
            nm = ~__builtin_amdgcn_perm(m, m, 0u);
            uint32_t gone = 0;
#pragma unroll
            for (int q = 0; q < Z; ++q) {
                uint32_t din[ND], dout[ND];
                read_row(din, kStage + (uint32_t)((2 * par) * Z + q) * kStaged + g4);
                read_row(dout, kStage + (uint32_t)((2 * par + 1) * Z + q) * kStaged + g4);
                e = (int)count_ge(din, nm, w, (uint32_t)e);
                gone = count_ge(dout, nm, w, gone);
            }
            e -= (int)gone;
            asm volatile("" : "+v"(e));
            if (kCoarse && !decltype(coarse)::value && par == 1) {
                asked = __builtin_amdgcn_readfirstlane((int)ask);
                asm volatile("" : "+s"(asked));
            }
            __syncthreads();
        };
        rows(
            y0, y1, wave, lane,
            [&](int y) {
                step(std::false_type{}, y, 0);
                step(std::false_type{}, y + 1, 1);
                more = max(more - 2 * kFar, 0);
                return asked != 0;
            },
            [&](int y) {
                step(std::true_type{}, y, 0);
                step(std::true_type{}, y + 1, 1);
            },
            [&](int n) {
                if (lane == 0) *(lds_u32*)(uintptr_t)(kKeep + 4 * wave) = more >= kFar * n / 2 ? 1u : 0u;
                more = 0;
            });
    }

    template <class Row>
    static __device__ __forceinline__ void slide(const Row& row, int W, int x0, int y0, int y1, int kh, int wave, int lane)
    {
        const int rx = KW / 2, ry = kh / 2;
        const uint32_t g4 = 4u * (uint32_t)(lane & (kGroups - 1));
        const int sub = P == 1 ? 0 : lane >> 5;
        auto gx_at = [&](int i) { return (uint32_t)min(max(x0 - rx + lane + i, 0), W - 1); };
        // first window, four rows at a time
        {
            uint32_t gx[NL], b[P][NL];
#pragma unroll
            for (int i = 0; i < NL; ++i) gx[i] = gx_at(64 * i);
            auto fetch = [&](int j) {
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    const int r = j + wave * P + q;
#pragma unroll
                    for (int i = 0; i < NL; ++i) b[q][i] = row(y0 - ry + r / Z, r % Z)[gx[i]];
                }
            };
            fetch(0);
            for (int j = 0; j < kh * Z; j += 4) {
#pragma unroll
                for (int q = 0; q < P; ++q)
#pragma unroll
                    for (int i = 0; i < NL; ++i)
                        *(lds_u8*)(uintptr_t)(kStage + (wave * P + q) * kStaged + lane + 64 * i) = (uint8_t)b[q][i];
                fetch(j + 4);
                __syncthreads();
                const int q = wave * P + sub;
                if (j + q < kh * Z) {
                    uint32_t d[1][ND];
                    read_row(d[0], kStage + q * kStaged + g4);
                    update<0, NG, false, false>(d, g4, 1);
                }
                __syncthreads();
            }
        }
        // Steps: half (columns [0, CH) or [CH, NG)) of the row that enters or
        // leaves is this wave's (P = 1) or half wave's (P = 2) to count.
        const int half = P == 1 ? wave & 1 : wave;
        const int leaves = P == 1 ? wave >> 1 : sub;
        // and this part of one row to stage
        const int frow = P == 1 ? wave >> 1 : wave, fx = P == 1 ? (wave & 1) * 64 * NF : 0;
        const int yoff = frow ? -ry : ry + 1;
        uint32_t gx[NF], buf[2][Z][NF];
#pragma unroll
        for (int i = 0; i < NF; ++i) gx[i] = gx_at(fx + 64 * i);
        auto fetch = [&](uint32_t (&b)[Z][NF], int y) {
#pragma unroll
            for (int q = 0; q < Z; ++q) {
                const unsigned char* p = row(y + yoff, q);
#pragma unroll
                for (int i = 0; i < NF; ++i) b[q][i] = p[gx[i]];
            }
        };
        auto put = [&](const uint32_t (&b)[Z][NF], int par) {
#pragma unroll
            for (int q = 0; q < Z; ++q)
#pragma unroll
                for (int i = 0; i < NF; ++i)
                    *(lds_u8*)(uintptr_t)(kStage + ((2 * par + frow) * Z + q) * kStaged + fx + lane + 64 * i) =
                        (uint8_t)b[q][i];
        };
        fetch(buf[0], y0);
        put(buf[0], 0);
        fetch(buf[1], y0 + 1);
        fetch(buf[0], y0 + 2);
        __syncthreads();
        uint32_t ask = 0;
        auto step = [&](auto coarse, int y, int par, uint32_t (&b)[Z][NF]) {
            uint32_t d[Z][ND];
#pragma unroll
            for (int q = 0; q < Z; ++q) read_row(d[q], kStage + (uint32_t)((2 * par + leaves) * Z + q) * kStaged + g4);
            put(b, par ^ 1);
            fetch(b, y + 3);
            const int one = leaves ? -1 : 1;
            if (half) update<CH, NG, true, decltype(coarse)::value>(d, g4, one);
            else update<0, CH, true, decltype(coarse)::value>(d, g4, one);
            if (kCoarse && !decltype(coarse)::value && par == 1) ask = *(const lds_u32*)(uintptr_t)kAsk;
            __syncthreads();
        };
        rows(
            y0, y1, kWaves + wave, lane,
            [&](int y) {
                step(std::false_type{}, y, 0, buf[1]);
                step(std::false_type{}, y + 1, 1, buf[0]);
                if constexpr (!kCoarse) return false;
                asm volatile("" : "+v"(ask));      // looked at after the barrier
                return __builtin_amdgcn_readfirstlane((int)ask) != 0;
            },
            [&](int y) {
                step(std::true_type{}, y, 0, buf[1]);
                step(std::true_type{}, y + 1, 1, buf[0]);
            },
            [](int) {});
    }
};

template <int KW, int P>
__global__ void __launch_bounds__(2 * 64 * kT / P)
mf_hist_kernel(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst, int H, int W, long long pitch,
               long long plane_stride, int ncol, int R, int kh)
{
    const int cb = (int)blockIdx.x % ncol, s = (int)blockIdx.x / ncol;
    const long long po = (long long)blockIdx.y * plane_stride;   // plane = blockIdx.y
    Hist<KW, P>::strip(src + po, dst + po, H, W, pitch, cb * Hist<KW, P>::kCols, s * R, min((s + 1) * R, H), kh);
}

// 3-D boxes, K x K x K: work-group row blockIdx.y is slice z0 + blockIdx.y.
template <int K, int P>
__global__ void __launch_bounds__(2 * 64 * kT / P)
mf_hist3_kernel(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst, int D, int H, int W,
                long long pitch, long long slice, int ncol, int R, int z0)
{
    typedef Hist<K, P, K> Box;
    const int cb = (int)blockIdx.x % ncol, s = (int)blockIdx.x / ncol, z = z0 + (int)blockIdx.y;
    Box::strip(src, dst + (long long)z * slice, H, W, pitch, cb * Box::kCols, s * R, min((s + 1) * R, H), K, D, slice, z);
}

// Rows of a block of the batched form: long enough that the first window
// (KW rows) is a small part, short enough that images of a few hundred rows
// still make several blocks.
constexpr int kBatchRows = 64;

template <int KW, int P>
__global__ void __launch_bounds__(2 * 64 * kT / P)
mf_hist_kernel_batched(const MfJob* __restrict__ jobs, int njobs, int nblocks)
{
    // not known to the compiler: it unrolls the first window's loops otherwise,
    // and keeps more addresses from block to block than two work-groups on a CU
    // have registers for
    int kh = KW;
    asm("" : "+s"(kh));
    for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
        int lo = 0, hi = njobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (jobs[mid].block_begin <= b) lo = mid;
            else hi = mid - 1;
        }
        const MfJob j = jobs[lo];
        const int lb = b - j.block_begin;
        const int y0 = lb / j.nbx * kBatchRows;
        Hist<KW, P>::strip(j.src, j.dst, j.H, j.W, j.pitch, lb % j.nbx * Hist<KW, P>::kCols, y0,
                           min(y0 + kBatchRows, j.H), kh);
        __syncthreads();   // the next block reuses the LDS
    }
}

template <int K, int P>
HistKernelInfo hist3_kernel()
{
    typedef Hist<K, P, K> Box;
    return {(const void*)mf_hist3_kernel<K, P>, nullptr, Box::kThreads, Box::kCols, 0, Box::kLds};
}

template <int KW, int P, bool BATCHED>
HistKernelInfo hist_kernel()
{
    typedef Hist<KW, P> Z;
    const void* b = nullptr;
    if constexpr (BATCHED) b = (const void*)mf_hist_kernel_batched<KW, P>;
    return {(const void*)mf_hist_kernel<KW, P>, b, Z::kThreads, Z::kCols, kBatchRows, Z::kLds};
}

}  // namespace
