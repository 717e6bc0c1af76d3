// What the cooperative solver kernels (cg_coop.hip, bicg_coop.hip) share: their
// launch, the words that cross blocks, and the columns of a block's rows.
//
// The kernels are launched as any other.  A grid has at most a block per CU of
// its stream, so its blocks come together as soon as what else runs on these
// CUs has ended; the first exchange waits for that, a few ms at most, and a
// launch that has waited in vain has changed nothing and is made again.  That
// happens when two such grids, of two threads or processes, are dispatched
// in the same few us and each holds CUs that the other needs: one in 1300
// solves of two processes that did nothing else.  (hipLaunchCooperativeKernel
// excludes it by a queue that the device gives to one process at a time, for
// tens of ms: with two processes on one card a CG solve of 25,600 rows took one
// of them 41 ms and the other 4.0, where alone it takes 1.0 and now takes both
// 1.14; 199,680 rows 144 and 2.6 ms, now 4.6 and 4.6; BiCGStab with three
// right-hand sides on 25,600 rows 54 and 6.0 ms, now 2.5 and 2.5.)
#pragma once
#include <algorithm>
#include <chrono>

#include "krylov.hpp"

namespace oasis {

namespace {

using u64 = unsigned long long;

constexpr int kCoopThreads = 1024;             // most threads of a block
constexpr int kCoopBlocks = 256;               // most blocks: four slots per lane of a reading wave
constexpr int kCoopMaxRows = kCoopBlocks * kCoopThreads;
constexpr int kBitWords = kCoopMaxRows / 32;
// The longest waits, in ticks of the 100 MHz wall clock: for the grid to come
// together 5 to 10 ms (of two grids that hold each other up one should give in
// well before the other), 2 s after that; and launches to come together in.
constexpr unsigned kJoinTicks = 500000, kCoopTicks = 200000000;
constexpr int kCoopTries = 6;

// The exchanged words: a T's bits, or the empty mark, a NaN that no sent
// value has (every NaN is sent as the quiet one).
template <typename T>
struct Word;
template <>
struct Word<float> {
    using U = unsigned;
    static constexpr U kEmpty = 0xffffbeefu, kNan = 0x7fc00000u;
    static __device__ __forceinline__ U of(float v) { return v == v ? __float_as_uint(v) : kNan; }
    static __device__ __forceinline__ float value(U u) { return __uint_as_float(u); }
};
template <>
struct Word<double> {
    using U = u64;
    static constexpr U kEmpty = 0xffffdeadbeef0001ull, kNan = 0x7ff8000000000000ull;
    static __device__ __forceinline__ U of(double v) {
        return v == v ? static_cast<U>(__double_as_longlong(v)) : kNan;
    }
    static __device__ __forceinline__ double value(U u) { return __longlong_as_double(static_cast<long long>(u)); }
};
template <typename U>
__device__ __forceinline__ U word_load(const U *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename U>
__device__ __forceinline__ void word_store(U *p, U v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// all of this wave's earlier stores have reached memory
__device__ __forceinline__ void stores_done() { __builtin_amdgcn_s_waitcnt(0x0f70); }   // vmcnt(0)

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// One step of wave_sums: M values over pairs of lanes (CTRL: the partner, BIT:
// what tells the two apart).  Of two values each lane keeps one and sends the
// other; the odd one out is summed in both.
template <int CTRL, int BIT, int M, int N>
__device__ __forceinline__ void sums_step(double (&v)[N]) {
    const bool up = (threadIdx.x >> BIT) & 1;
#pragma unroll
    for (int i = 0; i < M / 2; ++i) {
        const double a = v[2 * i], b = v[2 * i + 1];
        v[i] = (up ? b : a) + dpp_move<CTRL>(up ? a : b);
    }
    if constexpr (M % 2 != 0) v[M / 2] = v[M - 1] + dpp_move<CTRL>(v[M - 1]);
}

// v + v of the lane 16 (32) away
template <int ROWS>
__device__ __forceinline__ double across(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    if constexpr (ROWS == 1) {
        const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
    } else {
        const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        return __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
    }
}

// Sums over the wave of N <= 16 values (all lanes active): a lane gets that of
// value sums_index(), where that is below N.  Nine values take 80 instructions
// instead of 180 for nine wave_sum.
template <int N>
__device__ __forceinline__ double wave_sums(double (&v)[N]) {
    static_assert(N <= 16, "a row of lanes holds them");
    sums_step<kDppMirror, 3, N>(v);
    sums_step<kDppHalfMirror, 2, (N + 1) / 2>(v);
    sums_step<kDppXor3, 1, (N + 3) / 4>(v);
    sums_step<kDppXor1, 0, (N + 7) / 8>(v);
    return across<2>(across<1>(v[0]));
}
__device__ __forceinline__ int sums_index() {
    const int l = threadIdx.x & 15;
    return (l >> 3) | ((l >> 1) & 2) | ((l << 1) & 4) | ((l << 3) & 8);
}

// Halo entries (columns outside the block's rows) per thread at most.
template <int BS>
constexpr int kCoopHaloPer = BS >= 1024 ? 4 : 8;
// LDS of coop_columns.
constexpr size_t kCoopSetup = kBitWords * (sizeof(unsigned) + sizeof(unsigned short));

// Most blocks of a grid on this stream: one per CU that its kernels may use.
inline int coop_blocks(hipStream_t s, int *blocks) {
    int dev = 0, cu = 0;
    OASIS_TRY_HIP(hipGetDevice(&dev));
    OASIS_TRY_HIP(hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev));
    uint32_t mask[kCoopBlocks / 32] = {};
    int bits = 0;
    if (hipExtStreamGetCUMask(s, kCoopBlocks / 32, mask) == hipSuccess)
        for (uint32_t m : mask) bits += __builtin_popcount(m);
    else
        (void)hipGetLastError();
    if (bits > 0) cu = std::min(cu, bits);
    *blocks = std::min(cu, kCoopBlocks);
    return OASIS_OK;
}

// A launch's kJoinTicks to twice that.
inline unsigned join_ticks() {
    return kJoinTicks + static_cast<unsigned>(std::chrono::steady_clock::now().time_since_epoch().count() % kJoinTicks);
}

// The wait (1, 2, ...) that launch number `attempt` is to lose; see
// OASIS_KRYLOV_LOSE_WAIT.
inline int lose_wait(int lose, int attempt) { return attempt == 0 || (lose & 0x4000) ? lose & 0x3fff : 0; }

// This thread's row of the matrix (row `at` of [r0, r1)): its values, zero if
// it has no row (own), and its columns as positions in a block's vector of BS
// own entries followed by the halo's, two per word.  halo: the columns outside
// the block in ascending order; returns how many there are, and nothing else
// if they are more than fit.  mem: kCoopSetup bytes of LDS, free again on
// return; scan: a word per wave.
template <typename T, int BS>
__device__ __forceinline__ int coop_columns(int n, const EllCols &cols, const T *eval, int r0, int r1, int at, bool own,
                                            unsigned char *mem, int *halo, int *scan, T (&val)[kEll],
                                            unsigned (&idx)[kEll / 2]) {
    constexpr int E = kEll, WAVES = BS / kWave, MOST = kCoopHaloPer<BS> * BS;
    const int t = threadIdx.x, wv = t / kWave, wl = t & (kWave - 1);
    unsigned *bits = reinterpret_cast<unsigned *>(mem);
    unsigned short *rank = reinterpret_cast<unsigned short *>(mem + kBitWords * sizeof(unsigned));
    const int nw = (n + 31) / 32;
    for (int w = t; w < nw; w += BS) bits[w] = 0u;
    __syncthreads();
    int c[E];
    {
        const short *off = cols.offsets(at);
        const T *ev = eval + static_cast<size_t>(at) * kEll;
#pragma unroll
        for (int g = 0; g < E / 4; ++g) {
            const short4 d = *reinterpret_cast<const short4 *>(off + 4 * g);
            c[4 * g] = ell_col(at, d.x, n);
            c[4 * g + 1] = ell_col(at, d.y, n);
            c[4 * g + 2] = ell_col(at, d.z, n);
            c[4 * g + 3] = ell_col(at, d.w, n);
            T v[4];
            load4(ev + 4 * g, v);
#pragma unroll
            for (int k = 0; k < 4; ++k) val[4 * g + k] = own ? v[k] : T(0);
        }
    }
    if (own) {
#pragma unroll
        for (int k = 0; k < E; ++k)
            if (c[k] < r0 || c[k] >= r1) atomicOr(&bits[c[k] >> 5], 1u << (c[k] & 31));
    }
    __syncthreads();
    // ranks: halo entries in ascending column order
    int nh = 0;
    {
        constexpr int PER = kBitWords / BS;
        int cnt[PER], sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int w = t * PER + k;
            cnt[k] = w < nw ? __popc(bits[w]) : 0;
            sum += cnt[k];
        }
        int inc = sum;
        for (int o = 1; o < kWave; o <<= 1) {
            const int up = __shfl_up(inc, o, kWave);
            if (wl >= o) inc += up;
        }
        if (wl == kWave - 1) scan[wv] = inc;
        __syncthreads();
        int base = inc - sum;
        for (int w = 0; w < WAVES; ++w) {
            if (w < wv) base += scan[w];
            nh += scan[w];
        }
        nh = __builtin_amdgcn_readfirstlane(nh);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int w = t * PER + k;
            if (w < nw) {
                rank[w] = static_cast<unsigned short>(min(base, 65535));
                unsigned b = bits[w];
                int q = base;
                while (b) {
                    const int j = __builtin_ctz(b);
                    b &= b - 1;
                    if (q < MOST) halo[q] = w * 32 + j;
                    ++q;
                }
                base = q;
            }
        }
    }
    __syncthreads();
    if (nh > MOST) return nh;
#pragma unroll
    for (int k = 0; k < E; k += 2) {
        unsigned both[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int cc = c[k + q];
            const bool in = cc >= r0 && cc < r1;
            const int w = cc >> 5;
            const int h = in || !own ? 0 : rank[w] + __popc(bits[w] & ((1u << (cc & 31)) - 1u));
            both[q] = !own ? 0u : in ? cc - r0 : BS + h;
        }
        idx[k / 2] = both[0] | (both[1] << 16);
    }
    __syncthreads();
    return nh;
}

}  // namespace

}  // namespace oasis
