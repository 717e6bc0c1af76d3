// A run of CG iterations in one launch, for systems whose rows fit one per
// thread of a resident grid (at most 1024 rows per CU: 262,144 on gfx950).
//
// What bounds the two-kernel iteration at these sizes is not the matrix but
// the launches: on the 65x65x49 channel (199,680 rows, FP64) an iteration
// took 20 us in k_cg_p1_ell (12 us) and k_cg_p2 (6.4 us) and the gaps
// between them, against about 4 us that its 33 MB need at the cache rates; on the
// 1089-row Taylor-Green square each launch took 3.9 us for no work at all.
// Here a grid of blocks of up to 1024 threads, at most one per CU, keeps the
// matrix (values and local column indices) and the CG vectors in registers
// and each block's part of the direction, with the neighbours' entries it
// gathers, in LDS.  The recurrences are those of k_cg_p1 / k_cg_p2.
//
// An iteration has two grid-wide exchanges.  The first carries the new
// residual's entries and the partials of r.r together: with beta known,
// every block forms the direction of its own rows and of its halo (the
// columns its rows reference outside its range) by the same fused
// multiply-add, so the direction itself is never sent.  The second carries
// the partials of p.q.  A value that crosses blocks is one agent-scope
// atomic store into a slot that held the empty mark, and a reader polls the
// slot itself: no flag and no fence.  (An agent-scope fence writes back and
// invalidates the L2 and cost 38 us per barrier here; the polled exchange of
// two doubles between 256 blocks costs 1.5 us.  Words that carry a 32-bit
// number of the exchange beside 32 bits of payload need no emptying, but
// twice the polled words, and took 3.4 us.)
//
// An exchange has three buffers, used in turn by the iterations.  In
// iteration e a block empties its slots of iteration e + 2; they hold those
// of iteration e - 1, which every block has read, since all have sent a
// later exchange that this block has seen.  It waits for the emptying stores
// before it sends anything of iteration e + 1, so whoever polls for
// iteration e + 2, having seen all of e + 1, finds the slots empty or
// filled, never old.
//
// Every wait is bounded by the clock (coop.hpp).
//
// Per iteration, the kernel's duration by the iterations it ran (kernel trace),
// before and now: 65x65x49 FP64 20.0 -> 5.8 us (256 blocks, 780 rows each:
// about 1.7 us for each exchange, 0.4 us for the product, the rest block
// reductions, barriers and two divisions), FP32 with the null vector 12 -> 6.1
// us, 33x33x25 FP32 9.5 -> 5.0 us, 17x17x13 FP64 12 -> 4.0 us, a square of 2116
// rows 3.6 us, and by one block (k_cg_one) the one of 1089 rows 8 -> 2.5 us.
#include <algorithm>

#include "coop.hpp"

namespace oasis {

namespace {

struct CoopArgs {
    int n, rows;           // rows per block
    EllCols cols;
    const void *eval;
    const void *cur;       // RP pairs (r, p_old) entering iteration it0
    void *nxt[2];          // the pairs of either parity; (r, p) leave to that of the next iteration
    void *x;
    const void *wgt, *vnull;
    CGState *st;
    int it0, m, beta_zero;
    void *ex[3];           // exchanged residual entries, n words of T each
    u64 *slots[2];         // exchanged partials, first and second value
    unsigned join;         // ticks of the first wait
    int lose;              // the wait (1, 2, ...) that the last block takes as lost
};

// Partial slots of a value: [exchange kind][buffer][copy][block].  A block sends each value
// to eight copies and reads the one of its XCD: 256 readers of the same 2 KB
// wait for each other (2.5 us an exchange, 1.7 us with the copies).
constexpr int kCopies = kXcds;
constexpr int kSlotWords = 2 * 3 * kCopies * kCoopBlocks;
__device__ __forceinline__ int slot_set(int kind, int buf) { return (kind * 3 + buf) * kCopies * kCoopBlocks; }

// the state as k_cg_p1 and k_cg_p2 leave it; the flag of a block that lost its
// last wait outweighs the others'
__device__ __forceinline__ void leave(CGState *st, int flag, int it, double rr, double wrr, double rr_prev) {
    const int last = flag ? it : it - 1;   // the last iteration whose residual was seen
    if (flag) {
        atomicMax(&st->flag, flag);
        st->it_done = it;
        if (flag != 2) st->wrr = wrr;
    }
    if (!flag || flag == 2) {
        st->rr[last & 1] = rr;
        st->wrr_it = wrr;
        st->it_last = last;
    } else {
        st->rr[(it + 1) & 1] = rr_prev;
    }
}

// BS: threads of a block, and the most rows it has.
template <typename T, int BS>
__global__ __launch_bounds__(BS) void k_cg_coop(CoopArgs a) {
    constexpr int E = kEll;
    constexpr int kCoopWaves = BS / kWave;
    constexpr int kHaloPer = kCoopHaloPer<BS>, kCoopHalo = kHaloPer * BS;
    constexpr size_t kDir = (BS + kCoopHalo) * sizeof(T);
    // the bitmap of referenced columns (set-up) and the direction (iterations)
    __shared__ __align__(16) unsigned char shared[kCoopSetup > kDir ? kCoopSetup : kDir];
    __shared__ int halo[kCoopHalo];
    // [exchange kind][value]: the block's waves' sums and the grid's totals
    __shared__ double red[2][2][kCoopWaves], all[2][2];
    __shared__ int scan[kCoopWaves];
    __shared__ int quit;
    const int t = threadIdx.x, wv = t / kWave, wl = t & (kWave - 1);
    const int nb = gridDim.x, bid = blockIdx.x;
    const int r0 = bid * a.rows, r1 = min(a.n, r0 + a.rows);
    const int row = r0 + t;
    const bool own = row < r1;                 // this thread has a row
    const int at = own ? row : r0;             // a valid row for the loads
    CGState *st = a.st;
    if (t == 0) quit = 0;

    T val[E];
    unsigned idx[E / 2];
    const int nh = coop_columns<T, BS>(a.n, a.cols, static_cast<const T *>(a.eval), r0, r1, at, own, shared, halo, scan,
                                       val, idx);
    if (nh > kCoopHalo) {
        // not a system for this kernel: nothing has been sent, so no block
        // gets past its first exchange, and the host takes the other kernels
        if (t == 0) atomicMax(&st->flag, kCoopUnfit);
        return;
    }
    T *dir = reinterpret_cast<T *>(shared);

    const RP<T> *cur = static_cast<const RP<T> *>(a.cur);
    T *xg = static_cast<T *>(a.x);
    const T *vn = static_cast<const T *>(a.vnull);
    RP<T> me = cur[at];
    T x = xg[at];
    const double wgt = static_cast<double>(static_cast<const T *>(a.wgt)[at]);
    const T v = vn ? vn[at] : T(0);
    T r = me.r, p = a.beta_zero ? T(0) : me.p;
#pragma unroll
    for (int k = 0; k < kHaloPer; ++k) {
        const int h = t + k * BS;
        if (h < nh) dir[BS + h] = a.beta_zero ? T(0) : cur[halo[h]].p;
    }
    const double tol2 = st->tol2, upd2 = st->upd2;
    double rr_prev = st->rr[(a.it0 + 1) & 1];
    using W = Word<T>;
    using D = Word<double>;
    const int nv1 = vn ? 2 : 1;                // values of the second exchange

    // the end of an exchange, after the last poll of every wave: false when one
    // of them ran out
    int waits = 0;
    auto ended = [&]() -> bool {
        if (++waits == a.lose && bid == nb - 1 && t == 0) {
            atomicMax(&st->flag, waits == 1 ? kCoopLate : kCoopLost);
            quit = 1;
        }
        __syncthreads();
        return quit == 0;
    };
    // ask again, with the clock as a bound, while again() says so; the flag is
    // raised by whoever loses a wait first, not by those that it leaves behind
    auto poll = [&](auto &&again) {
        if (!again()) return;
        const unsigned began = static_cast<unsigned>(wall_clock64()), most = waits == 0 ? a.join : kCoopTicks;
        int k = 0;
        while (again()) {
            if ((++k & 63) != 0) continue;
            if (__hip_atomic_load(&st->flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= kCoopLate) {
                quit = 1;
                return;
            }
            if (static_cast<unsigned>(wall_clock64()) - began > most) {
                atomicMax(&st->flag, waits == 0 ? kCoopLate : kCoopLost);
                quit = 1;
                return;
            }
        }
    };
    int buf = 0, spare = 2;                    // buffers of this iteration and of the one after next
    // wave 0's slots: lanes 0..7 send the first value's copies, 8..15 the second's
    u64 *mine = (wl < kCopies ? a.slots[0] : a.slots[1]) + (wl & (kCopies - 1)) * kCoopBlocks + bid;
    const u64 *from0 = a.slots[0] + (bid & (kCopies - 1)) * kCoopBlocks + wl;
    const u64 *from1 = a.slots[1] + (bid & (kCopies - 1)) * kCoopBlocks + wl;
    // the block's sums of nv values, sent as its slots of an exchange
    auto give = [&](double s0, double s1, int nv, int kind) {
        s0 = wave_sum(s0);
        if (nv > 1) s1 = wave_sum(s1);
        if (wl == 0) {
            red[kind][0][wv] = s0;
            red[kind][1][wv] = s1;
        }
        __syncthreads();
        if (wv == 0) {
            const double u0 = row_sum(wl < kCoopWaves ? red[kind][0][wl] : 0.0);
            const double u1 = nv > 1 ? row_sum(wl < kCoopWaves ? red[kind][1][wl] : 0.0) : 0.0;
            if (wl < nv * kCopies) {
                word_store(mine + slot_set(kind, buf), D::of(wl < kCopies ? u0 : u1));
                word_store(mine + slot_set(kind, spare), D::kEmpty);
            }
        }
    };
    // every block's slots, read by wave 0 and summed in a fixed order; after
    // the next barrier the totals are in `all`
    auto take = [&](int nv, int kind) {
        if (wv != 0) return;
        constexpr int PER = kCoopBlocks / kWave;
        u64 u0[PER], u1[PER];
        const u64 *p0 = from0 + slot_set(kind, buf), *p1 = from1 + slot_set(kind, buf);
        poll([&] {
            bool miss = false;
#pragma unroll
            for (int k = 0; k < PER; ++k)
                if (wl + k * kWave < nb) {
                    u0[k] = word_load(p0 + k * kWave);
                    if (nv > 1) u1[k] = word_load(p1 + k * kWave);
                }
#pragma unroll
            for (int k = 0; k < PER; ++k)
                if (wl + k * kWave < nb) miss |= u0[k] == D::kEmpty || (nv > 1 && u1[k] == D::kEmpty);
            return miss;
        });
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (wl + k * kWave < nb) {
                s0 += D::value(u0[k]);
                if (nv > 1) s1 += D::value(u1[k]);
            }
        s0 = wave_sum(s0);
        if (nv > 1) s1 = wave_sum(s1);
        if (wl == 0) {
            all[kind][0] = s0;
            all[kind][1] = nv > 1 ? s1 : 0.0;
        }
    };

    int flag = 0, it = a.it0;
    double rr = 0.0, wrr = 0.0;
    for (; it < a.it0 + a.m; ++it) {
        typename W::U *ex = static_cast<typename W::U *>(a.ex[buf]);
        stores_done();
        if (own) {
            word_store(static_cast<typename W::U *>(a.ex[spare]) + row, W::kEmpty);
            word_store(ex + row, W::of(r));
        }
        const double rd = r;
        give(own ? rd * rd : 0.0, own ? wgt * rd * rd : 0.0, 2, 0);
        typename W::U hw[kHaloPer];
        poll([&] {
            bool miss = false;
#pragma unroll
            for (int k = 0; k < kHaloPer; ++k) {
                const int h = t + k * BS;
                if (h < nh) hw[k] = word_load(ex + halo[h]);
            }
#pragma unroll
            for (int k = 0; k < kHaloPer; ++k)
                if (t + k * BS < nh) miss |= hw[k] == W::kEmpty;
            return miss;
        });
        take(2, 0);
        if (!ended()) break;
        rr = all[0][0];
        wrr = all[0][1];
        if (!finite(wrr) || !finite(rr))
            flag = 3;
        else if (wrr <= tol2)
            flag = 1;
        else if (wrr <= upd2)
            flag = 4;
        if (flag) break;
        const bool fresh = a.beta_zero && it == a.it0;
        const T beta = fresh ? T(0) : static_cast<T>(rr / rr_prev);
        rr_prev = rr;
        p = fresh ? r : fma_t(beta, p, r);
        if (own) dir[t] = p;
#pragma unroll
        for (int k = 0; k < kHaloPer; ++k) {
            const int h = t + k * BS;
            if (h < nh) {
                const T rh = W::value(hw[k]);
                dir[BS + h] = fresh ? rh : fma_t(beta, dir[BS + h], rh);
            }
        }
        __syncthreads();
        T q = T(0);
#pragma unroll
        for (int k = 0; k < E; k += 2) {
            q += val[k] * dir[idx[k / 2] & 0xffffu];
            q += val[k + 1] * dir[idx[k / 2] >> 16];
        }
        give(own ? static_cast<double>(p) * static_cast<double>(q) : 0.0,
             own ? static_cast<double>(v) * static_cast<double>(q) : 0.0, nv1, 1);
        take(nv1, 1);
        if (!ended()) break;
        const double pq = all[1][0], vq = all[1][1];
        if (!(pq > 0.0) || !finite(pq)) {
            flag = finite(pq) ? 2 : 3;
            break;
        }
        const T al = static_cast<T>(rr / pq), cv = static_cast<T>(vq);
        x += al * p;
        r -= al * (vn ? q - cv * v : q);
        spare = buf;
        buf = buf == 2 ? 0 : buf + 1;
    }
    if (quit) return;
    if (own) {
        xg[row] = x;
        static_cast<RP<T> *>(a.nxt[it & 1])[row] = RP<T>{r, p};
    }
    if (bid == 0 && t == 0) leave(st, flag, it, rr, wrr, rr_prev);
}


// The same run by one block, R rows a thread, for systems that fit it: what
// the blocks exchange lies in LDS, and an iteration is two block sums and
// three barriers.  1089 rows of 7 entries, FP64: an iteration took 3.7 us of a
// solve by five blocks, 2.7 by one (3.5 with the padding's gathers); the limit
// is the registers of two rows.
constexpr int kOneThreads = 1024, kOneRows = 2;
template <typename T, int R>
__global__ __launch_bounds__(kOneThreads) void k_cg_one(CoopArgs a) {
    constexpr int E = kEll, WAVES = kOneThreads / kWave;
    __shared__ T dir[R * kOneThreads];
    __shared__ double red[2][2][WAVES];   // [sum][value]: the waves' parts
    const int t = threadIdx.x, wv = t / kWave, wl = t & (kWave - 1);
    CGState *st = a.st;
    const RP<T> *cur = static_cast<const RP<T> *>(a.cur);
    T *xg = static_cast<T *>(a.x);
    const T *vn = static_cast<const T *>(a.vnull);
    T val[R][E], x[R], r[R], p[R], v[R];
    double wgt[R];
    unsigned idx[R][E / 2];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int row = t + k * kOneThreads;
        const bool own = row < a.n;
        const int at = own ? row : 0;
        const short *off = a.cols.offsets(at);
        const T *ev = static_cast<const T *>(a.eval) + static_cast<size_t>(at) * kEll;
#pragma unroll
        for (int g = 0; g < E / 4; ++g) {
            const short4 d = *reinterpret_cast<const short4 *>(off + 4 * g);
            T w[4];
            load4(ev + 4 * g, w);
#pragma unroll
            for (int q = 0; q < 4; ++q) val[k][4 * g + q] = own ? w[q] : T(0);
            idx[k][2 * g] = static_cast<unsigned>(ell_col(at, d.x, a.n) | ell_col(at, d.y, a.n) << 16);
            idx[k][2 * g + 1] = static_cast<unsigned>(ell_col(at, d.z, a.n) | ell_col(at, d.w, a.n) << 16);
        }
        const RP<T> me = cur[at];
        // a thread without a row has zeros throughout
        x[k] = own ? xg[at] : T(0);
        r[k] = own ? me.r : T(0);
        p[k] = own && !a.beta_zero ? me.p : T(0);
        v[k] = own && vn ? vn[at] : T(0);
        wgt[k] = own ? static_cast<double>(static_cast<const T *>(a.wgt)[at]) : 0.0;
    }
    // pairs of entries that some row has: 8 of 16 slots are padding in 2D, and
    // the gathers from LDS are half of an iteration
    __shared__ int pairs[WAVES];
    int np = 0;
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (__ballot(val[k][e] != T(0))) np = e / 2 + 1;
    if (wl == 0) pairs[wv] = np;
    __syncthreads();
    for (int w = 0; w < WAVES; ++w) np = max(np, pairs[w]);
    np = __builtin_amdgcn_readfirstlane(np);
    const double tol2 = st->tol2, upd2 = st->upd2;
    double rr_prev = st->rr[(a.it0 + 1) & 1];
    // the block's sums in every thread, in a fixed order
    auto total = [&](double &s0, double &s1, int kind) {
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        if (wl == 0) {
            red[kind][0][wv] = s0;
            red[kind][1][wv] = s1;
        }
        __syncthreads();
        s0 = row_sum(red[kind][0][wl & (WAVES - 1)]);
        s1 = row_sum(red[kind][1][wl & (WAVES - 1)]);
    };
    static_assert(WAVES == 16, "a row of lanes holds the waves' parts");

    int flag = 0, it = a.it0;
    double rr = 0.0, wrr = 0.0;
    for (; it < a.it0 + a.m; ++it) {
        rr = wrr = 0.0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const double rd = r[k];
            rr += rd * rd;
            wrr += wgt[k] * rd * rd;
        }
        total(rr, wrr, 0);
        if (!finite(wrr) || !finite(rr))
            flag = 3;
        else if (wrr <= tol2)
            flag = 1;
        else if (wrr <= upd2)
            flag = 4;
        if (flag) break;
        const bool fresh = a.beta_zero && it == a.it0;
        const T beta = fresh ? T(0) : static_cast<T>(rr / rr_prev);
        rr_prev = rr;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            p[k] = fresh ? r[k] : fma_t(beta, p[k], r[k]);
            dir[t + k * kOneThreads] = p[k];
        }
        __syncthreads();
        T q[R];
        double pq = 0.0, vq = 0.0;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            q[k] = T(0);
#pragma unroll
            for (int e = 0; e < E; e += 2) {
                if (e / 2 >= np) break;
                unsigned both = idx[k][e / 2];
                asm volatile("" : "+v"(both));   // unpacked here, not once into 16 registers
                q[k] += val[k][e] * dir[both & 0xffffu];
                q[k] += val[k][e + 1] * dir[both >> 16];
            }
            pq += static_cast<double>(p[k]) * static_cast<double>(q[k]);
            vq += static_cast<double>(v[k]) * static_cast<double>(q[k]);
        }
        total(pq, vq, 1);
        if (!(pq > 0.0) || !finite(pq)) {
            flag = finite(pq) ? 2 : 3;
            break;
        }
        const T al = static_cast<T>(rr / pq), cv = static_cast<T>(vq);
#pragma unroll
        for (int k = 0; k < R; ++k) {
            x[k] += al * p[k];
            r[k] -= al * (vn ? q[k] - cv * v[k] : q[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int row = t + k * kOneThreads;
        if (row < a.n) {
            xg[row] = x[k];
            static_cast<RP<T> *>(a.nxt[it & 1])[row] = RP<T>{r[k], p[k]};
        }
    }
    if (t == 0) leave(st, flag, it, rr, wrr, rr_prev);
}

// every exchange slot empty, and no flag
template <typename T>
__global__ __launch_bounds__(kBlock) void k_words_clear(int n, CoopArgs a) {
    using W = Word<T>;
    const int step = gridDim.x * blockDim.x, i0 = blockIdx.x * blockDim.x + threadIdx.x;
    for (int k = 0; k < 3; ++k)
        for (int i = i0; i < n; i += step) static_cast<typename W::U *>(a.ex[k])[i] = W::kEmpty;
    for (int i = i0; i < kSlotWords; i += step) a.slots[0][i] = a.slots[1][i] = Word<double>::kEmpty;
    if (i0 == 0) a.st->flag = 0;
}

}  // namespace

namespace {

// *most = the widest halo of the blocks of `rows` rows, from the ELL offsets
__global__ __launch_bounds__(kCoopThreads) void k_coop_halo(int n, int rows, const short *__restrict__ ecol, int *most) {
    __shared__ unsigned bits[kBitWords];
    __shared__ int count;
    const int t = threadIdx.x, r0 = blockIdx.x * rows, r1 = min(n, r0 + rows), nw = (n + 31) / 32;
    for (int w = t; w < nw; w += kCoopThreads) bits[w] = 0u;
    if (t == 0) count = 0;
    __syncthreads();
    constexpr int Q = kEll / 4;               // four offsets at a time
    for (int i = r0 * Q + t; i < r1 * Q; i += kCoopThreads) {
        const short4 d = reinterpret_cast<const short4 *>(ecol)[i];
        const int row = i / Q;
        const int c[4] = {ell_col(row, d.x, n), ell_col(row, d.y, n), ell_col(row, d.z, n), ell_col(row, d.w, n)};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c[k] < r0 || c[k] >= r1) atomicOr(&bits[c[k] >> 5], 1u << (c[k] & 31));
    }
    __syncthreads();
    int mine = 0;
    for (int w = t; w < nw; w += kCoopThreads) mine += __popc(bits[w]);
    if (mine) atomicAdd(&count, mine);
    __syncthreads();
    if (t == 0 && count) atomicMax(most, count);
}

}  // namespace

int coop_halo(hipStream_t s, int n, const short *ecol, int *most, int *room) {
    int blocks = 0;
    *room = 0;
    OASIS_TRY(coop_blocks(s, &blocks));
    if (n > blocks * kCoopThreads) return OASIS_OK;
    const int grid = std::min(blocks, (n + kBlock - 1) / kBlock), rows = (n + grid - 1) / grid;
    *room = rows <= 256 ? kCoopHaloPer<256> * 256 : rows <= 512 ? kCoopHaloPer<512> * 512 : kCoopHaloPer<1024> * 1024;
    if (n - rows <= *room) return OASIS_OK;   // whatever the columns are
    hipLaunchKernelGGL(k_coop_halo, dim3(grid), dim3(kCoopThreads), 0, s, n, rows, ecol, most);
    OASIS_TRY_LAUNCH();
    return OASIS_OK;
}

template <typename T>
bool cg_coop_fits(hipStream_t s, int n, CGWork<T> &w) {
    // one row per thread of one block per CU; the kernel and grid the caller
    // asked for by name are left as they are
    if (!w.cols.any() || !w.eval || !w.tun.ell() || w.tun.cg_form != OASIS_CG_FORM_AUTO ||
        !w.tun.grid_auto || n > kCoopMaxRows)
        return false;
    int most = 0;
    return coop_blocks(s, &most) == OASIS_OK && n <= most * kCoopThreads && w.coop.next();
}

template <typename T>
int cg_coop_run(hipStream_t s, int n, CGWork<T> &w, T *x, const T *wgt, const T *vnull, int it0, int m, bool beta_zero,
                CGState *h, int *lost) {
    int most = 0;
    OASIS_TRY(coop_blocks(s, &most));
    // as many blocks as there are, down to 256 rows each: fewer rows per
    // block shorten the gathers, and the exchange hardly depends on the grid
    // (1.4 us between 32 blocks, 1.5 us between 256)
    const int grid = std::min(most, (n + kBlock - 1) / kBlock);
    CoopArgs a{};
    a.n = n;
    a.rows = (n + grid - 1) / grid;
    a.cols = w.cols;
    a.eval = w.eval;
    a.cur = w.pair[it0 & 1];
    // the exchanged words live in the second halves of the two CG records
    // (the pairs use the first ones) and in the partial arrays, which this
    // form does not use
    for (int k = 0; k < 2; ++k) a.nxt[k] = w.pair[k];
    a.ex[0] = reinterpret_cast<T *>(w.pair[0] + n);
    a.ex[1] = reinterpret_cast<T *>(w.pair[0] + n) + n;
    a.ex[2] = reinterpret_cast<T *>(w.pair[1] + n);
    a.x = x;
    a.wgt = wgt;
    a.vnull = vnull;
    a.st = w.st;
    a.it0 = it0;
    a.m = m;
    a.beta_zero = beta_zero ? 1 : 0;
    a.slots[0] = reinterpret_cast<u64 *>(w.partA);
    a.slots[1] = reinterpret_cast<u64 *>(w.partB);
    if (n <= kOneThreads * kOneRows) {
        if (n <= kOneThreads)
            hipLaunchKernelGGL((k_cg_one<T, 1>), dim3(1), dim3(kOneThreads), 0, s, a);
        else
            hipLaunchKernelGGL((k_cg_one<T, kOneRows>), dim3(1), dim3(kOneThreads), 0, s, a);
        OASIS_TRY_LAUNCH();
        return read_state(s, w.stage, w.st, h, sizeof(*h));
    }
    void *args[] = {&a};
    const void *kern;
    int bs;
    if (a.rows <= 256) {
        kern = reinterpret_cast<const void *>(&k_cg_coop<T, 256>);
        bs = 256;
    } else if (a.rows <= 512) {
        kern = reinterpret_cast<const void *>(&k_cg_coop<T, 512>);
        bs = 512;
    } else {
        kern = reinterpret_cast<const void *>(&k_cg_coop<T, 1024>);
        bs = 1024;
    }
    for (int attempt = 0;; ++attempt) {
        a.join = join_ticks();
        a.lose = lose_wait(w.lose, attempt);
        hipLaunchKernelGGL(k_words_clear<T>, dim3(grid_for(n, kBlock, 1024)), dim3(kBlock), 0, s, n, a);
        OASIS_TRY_LAUNCH();
        if (hipLaunchKernel(kern, dim3(grid), dim3(bs), args, 0, s) != hipSuccess) {
            // refused (nothing has run): the caller takes the other kernels
            (void)hipGetLastError();
            return OASIS_EUNSUPPORTED;
        }
        OASIS_TRY(read_state(s, w.stage, w.st, h, sizeof(*h)));
        if (h->flag < kCoopLate) return OASIS_OK;
        *lost += 1;
        // (a later wait is lost after blocks may have written x)
        if (h->flag != kCoopLate || attempt + 1 == kCoopTries) return OASIS_OK;
    }
}

template bool cg_coop_fits<double>(hipStream_t, int, CGWork<double> &);
template bool cg_coop_fits<float>(hipStream_t, int, CGWork<float> &);
template int cg_coop_run<double>(hipStream_t, int, CGWork<double> &, double *, const double *, const double *, int,
                                 int, bool, CGState *, int *);
template int cg_coop_run<float>(hipStream_t, int, CGWork<float> &, float *, const float *, const float *, int, int,
                                bool, CGState *, int *);

}  // namespace oasis
