// A whole BiCGStab solve in one launch, for systems whose rows fit one per
// thread of a resident grid (at most 1024 rows per CU: 262,144 on gfx950).
//
// At these sizes the kernels of an iteration are launches rather than work:
// three of 5-6 us on the 1089-row Taylor-Green square, about 14 us each on
// 90,000 rows, and each convergence test that stops one right-hand side, the
// explicit residual that confirms it and the resumption cost the host a
// read-back of 20 us or more besides.  Here a cooperative grid keeps the
// matrix (values and local column indices) and the vectors r, u, v and r_hat
// of all right-hand sides in registers and the block's part of the
// vector to be multiplied, with the neighbours' entries, in LDS; the tests,
// confirmations and restarts run inside it.  The recurrences, the tests and
// their order are those of k_bi_1, k_bi_2 and k_bi_3 and of the host's loop
// around them.
//
// Two exchanges make up an iteration's traffic, each a polled word (coop.hpp):
// - the vector to be multiplied (x, p, s): its entries go to words that the
//   blocks whose halo they are in poll; three sets of words, used in turn;
// - the sums: every block sends its partials and reads everybody's; four
//   sets of slots, used in turn.
// A vector is never sent twice without a sum between them.
//
// Slots of sum e are emptied in sum e + 2: this block has then seen all of
// e + 1, which a block sends after it has read all of e.  They serve sum
// e + 4, and the emptying has reached memory before this block sends
// anything of e + 3, which every reader of e + 4 has seen.  Words of vector e
// are emptied with vector e + 1: between the two lies a sum that every block
// has sent after it read its halo of e.  They serve vector e + 3, and the
// emptying has reached memory before this block sends vector e + 2 and hence
// its part of the sum that follows it.
//
// Every wait is bounded by the clock (coop.hpp).  A block that has lost one
// sends nothing more, and the host puts the start iterate back before the solve
// is begun again: blocks that got further may have moved their part of x.
//
// The kernel's duration by its iterations, with three right-hand sides in FP64
// (kernel trace; the set-up of its columns and the confirmations are in it):
// 199,680 rows 39 us of 64 iterations (product 9, halo 9, sums 14, scalars and
// updates 4, barriers; three kernels of 42 and the read-backs before it: 75),
// 3264 rows 17 us of 25; with one right-hand side 17 and 11.5.  The velocity
// phase of a time step whose iteration cap lets it come here (kCoopRun) went
// from 1650 to 900 us on 199,680 rows, from 1110 to 540 on 105,000, from 670 to 300
// on 3264 (the first of two solves), and from 460 to 146 on the 1089-row
// square.
// Nine sums by one exchange of lanes (coop.hpp's wave_sums) took 3.5 us of an
// iteration where nine wave sums took 7; vector words by right-hand side, not
// by row, 8 us where rows of three took 17; the scalars in lane k, not in all,
// 4 us where they took up to 14.
#include <algorithm>

#include "coop.hpp"

namespace oasis {

namespace {

// c - a b in one rounding (the form of k_bi_2 and k_bi_3)
template <typename T>
__device__ __forceinline__ T fms_t(T c, T a, T b) {
    return fma_t(-a, b, c);
}

// p[i], by a 32-bit byte offset from a base that every lane has.  (The
// offset is hidden so that the sum is not kept in two registers per base.)
template <typename T>
__device__ __forceinline__ T &item(const void *p, unsigned bytes) {
    asm volatile("" : "+v"(bytes));
    return *reinterpret_cast<T *>(static_cast<char *>(const_cast<void *>(p)) + bytes);
}

struct BiCoopArgs {
    int n, rows;           // rows per block
    EllCols cols;
    const void *eval;
    const void *wgt;
    const void *b[3];
    void *x[3];
    void *keep_s[3], *keep_t[3];   // s and t while an explicit residual is formed at the s stage
    void *v[3], *rhat[3];          // where these are in memory (LEAN)
    void *x0;              // the start iterate, [NR][n] (not inner)
    BiBlock *blk;          // results, and glob.pause: kCoopLate to kCoopUnfit
    double rtol2;
    int maxit, inner;
    void *ex[3];           // sets of vector words, [NR][n] of T each
    u64 *slots;            // four sets of [value][copy][block]
    int copies;            // of a slot, read by the XCDs in turn
    unsigned join;         // ticks of the first wait
    int lose;              // the wait (1, 2, ...) that the last block takes as lost
};

// BS: threads of a block, and the most rows it has.
template <typename T, int NR, int BS>
__global__ __launch_bounds__(BS) void k_bi_coop(BiCoopArgs a) {
    constexpr int E = kEll, WAVES = BS / kWave, NV = 3 * NR;
    constexpr int PER = kCoopHaloPer<BS>, HALO = PER * BS, LEN = BS + HALO;
    constexpr bool LEAN = BS >= 1024 && sizeof(T) * NR > 8;   // two more vectors in memory
    constexpr int CHUNK = LEAN && NR == 3 ? 2 : PER;          // halo entries polled together
    constexpr size_t kVec = (size_t)NR * LEN * sizeof(T);
    __shared__ __align__(16) unsigned char shared[kCoopSetup > kVec ? kCoopSetup : kVec];
    __shared__ int halo[HALO];
    __shared__ double red[NV][WAVES], all[NV];    // the waves' sums, the grid's
    __shared__ double scal[WAVES][6 * NR];
    __shared__ BiState result[NR];
    __shared__ int scan[WAVES];
    // a wait of a sum, of a product, was lost: two, so that a wave still at the
    // test of one cannot see what a wave ahead of it sets in the next
    __shared__ int quit[2];
    constexpr int kTold = 1, kRanOut = 2;         // by the flag; by the clock
    const int t = threadIdx.x, wv = t / kWave, wl = t & (kWave - 1);
    const int nb = gridDim.x, bid = blockIdx.x;
    const int r0 = bid * a.rows, r1 = min(a.n, r0 + a.rows);
    const int row = r0 + t;
    const bool own = row < r1;                    // this thread has a row
    const int at = own ? row : min(r0, a.n - 1);  // a valid row for the loads
    int *flag = &a.blk->glob.pause;
    if (t < 2) quit[t] = 0;

    T val[E];
    unsigned idx[E / 2];
    const int nh = coop_columns<T, BS>(a.n, a.cols, static_cast<const T *>(a.eval), r0, r1, at, own, shared, halo, scan,
                                       val, idx);
    if (nh > HALO) {
        // not a system for this kernel: nothing has been sent, so no block
        // gets past its first sum, and the host takes the other kernels
        if (t == 0) atomicMax(flag, kCoopUnfit);
        return;
    }
    T *vec = reinterpret_cast<T *>(shared);       // [NR][LEN]: own entries, then the halo's
    using W = Word<T>;
    using D = Word<double>;

    // the end of an exchange, after the last poll of every wave: false when one
    // of them ran out
    int waits = 0;
    auto ended = [&](int kind) -> bool {
        if (++waits == a.lose && bid == nb - 1 && t == 0) quit[kind] = kRanOut;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(quit[kind]) == 0;
    };
    // ask again, with the clock as a bound, while again() says so
    auto poll = [&](int kind, auto &&again) {
        if (!again()) return;
        const unsigned began = static_cast<unsigned>(wall_clock64()), most = waits == 0 ? a.join : kCoopTicks;
        int k = 0;
        while (again()) {
            if ((++k & 63) != 0) continue;
            const bool told = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= kCoopLate;
            if (told || static_cast<unsigned>(wall_clock64()) - began > most) {
                quit[kind] = told ? kTold : kRanOut;
                return;
            }
        }
    };
    // all[j] = the grid's sum of c[j] for j < nv, added in a fixed order; false
    // when a wait ran out
    const int set = NV * a.copies * nb;
    int sum_set = 0;
    auto total = [&](double (&c)[NV], int nv) -> bool {
#pragma unroll
        for (int j = 0; j < NV; ++j) c[j] = own ? c[j] : 0.0;
        const double sums = wave_sums<NV>(c);
        if (wl < 16 && sums_index() < nv) red[sums_index()][wv] = sums;
        stores_done();
        __syncthreads();
        u64 *to = a.slots + sum_set * set + wl * nb + bid, *spare = a.slots + ((sum_set + 2) & 3) * set + wl * nb + bid;
        for (int j = wv; j < NV; j += WAVES) {
            if (j < nv) {
                const double s = row_sum(wl < WAVES ? red[j][wl] : 0.0);
                if (wl < a.copies) word_store(to + j * a.copies * nb, D::of(s));
            }
            if (wl < a.copies) word_store(spare + j * a.copies * nb, D::kEmpty);
        }
        const u64 *from = a.slots + sum_set * set + (bid % kXcds % a.copies) * nb + wl;
        for (int j = wv; j < nv; j += WAVES) {
            constexpr int SL = kCoopBlocks / kWave;
            u64 u[SL];
            const u64 *f = from + j * a.copies * nb;
            poll(0, [&] {
                bool miss = false;
#pragma unroll
                for (int k = 0; k < SL; ++k)
                    if (wl + k * kWave < nb) u[k] = word_load(f + k * kWave);
#pragma unroll
                for (int k = 0; k < SL; ++k)
                    if (wl + k * kWave < nb) miss |= u[k] == D::kEmpty;
                return miss;
            });
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < SL; ++k)
                if (wl + k * kWave < nb) s += D::value(u[k]);
            s = wave_sum(s);
            if (wl == 0) all[j] = s;
        }
        sum_set = (sum_set + 1) & 3;
        return ended(0);
    };
    // q = As m: the vectors m go to the words and into LDS with their halo;
    // false when a wait ran out (q is not to be used then)
    int vec_set = 0;
    auto product = [&](const T(&m)[NR], T(&q)[NR]) -> bool {
        using U = typename W::U;
        void *ex = a.ex[vec_set], *spare = a.ex[vec_set == 0 ? 2 : vec_set - 1];
        const unsigned mine = static_cast<unsigned>(row) * sizeof(T), plane = static_cast<unsigned>(a.n) * sizeof(T);
        stores_done();
        if (own) {
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                word_store(&item<U>(ex, mine + k * plane), W::of(m[k]));
                vec[k * LEN + t] = m[k];
            }
#pragma unroll
            for (int k = 0; k < NR; ++k) word_store(&item<U>(spare, mine + k * plane), W::kEmpty);
        }
#pragma unroll
        for (int h0 = 0; h0 < PER; h0 += CHUNK) {
            U hw[CHUNK][NR];
            poll(1, [&] {
                bool miss = false;
#pragma unroll
                for (int h = 0; h < CHUNK; ++h)
                    if (t + (h0 + h) * BS < nh) {
                        const unsigned p = static_cast<unsigned>(halo[t + (h0 + h) * BS]) * sizeof(T);
#pragma unroll
                        for (int k = 0; k < NR; ++k) hw[h][k] = word_load(&item<U>(ex, p + k * plane));
                    }
#pragma unroll
                for (int h = 0; h < CHUNK; ++h)
                    if (t + (h0 + h) * BS < nh) {
#pragma unroll
                        for (int k = 0; k < NR; ++k) miss |= hw[h][k] == W::kEmpty;
                    }
                return miss;
            });
#pragma unroll
            for (int h = 0; h < CHUNK; ++h)
                if (t + (h0 + h) * BS < nh) {
#pragma unroll
                    for (int k = 0; k < NR; ++k) vec[k * LEN + BS + t + (h0 + h) * BS] = W::value(hw[h][k]);
                }
        }
        vec_set = vec_set == 2 ? 0 : vec_set + 1;
        if (!ended(1)) return false;
#pragma unroll
        for (int k = 0; k < NR; ++k) q[k] = T(0);
#pragma unroll
        for (int e = 0; e < E; e += 2) {
            unsigned both = idx[e / 2];
            asm volatile("" : "+v"(both));        // unpacked here, not once into 16 registers
            const unsigned i0 = both & 0xffffu, i1 = both >> 16;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                q[k] += val[e] * vec[k * LEN + i0];
                q[k] += val[e + 1] * vec[k * LEN + i1];
            }
        }
        return true;
    };
    const double wd = static_cast<double>(item<const T>(a.wgt, static_cast<unsigned>(at) * sizeof(T)));
    const unsigned off = static_cast<unsigned>(at) * sizeof(T);
    auto rhs = [&](int k) { return item<const T>(a.b[k], off); };
    // x stays in memory, and s and t go there over kExit's product: 128
    // registers a thread is what 1024 threads have
    auto xk = [&](int k) -> T & { return item<T>(a.x[k], off); };
    T r[NR], u[NR], vr[NR], hr[NR];
    auto vk = [&](int k) -> T {
        if constexpr (LEAN) return item<const T>(a.v[k], off);
        return vr[k];
    };
    auto hk = [&](int k) -> T {
        if constexpr (LEAN) return item<const T>(a.rhat[k], off);
        return hr[k];
    };
    auto set_v = [&](int k, T value) {
        if constexpr (!LEAN)
            vr[k] = value;
        else if (own)
            item<T>(a.v[k], off) = value;
    };
    auto set_h = [&](int k, T value) {
        if constexpr (!LEAN)
            hr[k] = value;
        else if (own)
            item<T>(a.rhat[k], off) = value;
    };
    // The wave's copy of the scalars: rho, alpha, omega of the last iteration,
    // the tolerance, r_hat.r entering this one and its beta.  Lane k works out
    // those of right-hand side k; in registers of every lane they cost 40
    // registers and three times the divisions.
    constexpr int kRho = 0, kAlpha = NR, kOmega = 2 * NR, kTol2 = 3 * NR, kRr = 4 * NR, kBeta = 5 * NR;
    const int lk = wl < NR ? wl : 0;
    auto get = [&](int i) { return scal[wv][i]; };
    auto put = [&](int i, double value) {         // value of lane k in entry i + k
        if (wl < NR) scal[wv][i + wl] = value;
        wave_lds_sync();
    };
    // the right-hand sides for which a condition holds in their lane
    auto those = [&](bool c) { return static_cast<int>(__ballot(wl < NR && c)); };
    int again[NR], no_sexit[NR];                  // restarts and refused candidates; see BiState
    int active = (1 << NR) - 1, restarted = 0, it = 0;
    auto done = [&](int k, int status, int iters, double w2) {
        active &= ~(1 << k);
        if (t == 0) {
            result[k].event = status;
            result[k].it_rec = iters;
            result[k].wrr_rec = w2;
            result[k].active = again[k];
        }
    };
    auto restart = [&](int k) -> bool {           // from r itself; once
        if ((restarted >> k) & 1) {
            done(k, OASIS_EBREAKDOWN, it, -1.0);
            return false;
        }
        restarted |= 1 << k;
        again[k] += 1;
        if (wl == 0) scal[wv][kRho + k] = scal[wv][kAlpha + k] = scal[wv][kOmega + k] = 1.0;
        wave_lds_sync();
        u[k] = T(0);
        set_h(k, r[k]);
        return true;
    };
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        if (a.inner && own) xk(k) = T(0);
        again[k] = 0;
        no_sexit[k] = -1;
        u[k] = T(0);
        r[k] = rhs(k);
    }
    put(kRho, 1.0);
    put(kAlpha, 1.0);
    put(kOmega, 1.0);

    // One product and one sum a turn; what they are of depends on the step:
    //   kStart  the first residual          kCheck, kCap  b - As x of candidates, of all at the last iteration
    //   kNorms  no product: the residuals   kP  p = r + beta u and v = As p
    //   kS      s = r - alpha v and As s    kExit  b - As (x + alpha p) of candidates at the s stage
    enum { kStart, kCheck, kCap, kNorms, kP, kS, kExit };
    int step = kStart, cands = 0;
    while (true) {
        T q[NR];
        if (step != kNorms && !(step == kStart && a.inner)) {
            T m[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                if (step == kP)
                    m[k] = fma_t(static_cast<T>(get(kBeta + k)), u[k], r[k]);
                else if (step == kS)
                    m[k] = r[k];
                else if (step == kExit)
                    m[k] = xk(k) + static_cast<T>(get(kAlpha + k)) * u[k];
                else
                    m[k] = xk(k);
            }
            if (!product(m, q)) break;
        }
        // (one call of total: its code in one place stays in the instruction cache)
        double c[NV];
        int nv = NR;
#pragma unroll
        for (int j = 0; j < NV; ++j) c[j] = 0.0;
        if (step == kP) {
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                set_v(k, q[k]);
                c[k] = static_cast<double>(hk(k)) * static_cast<double>(q[k]);
            }
        } else if (step == kS) {
            nv = 3 * NR;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                r[k] = vec[k * LEN + t];          // s
                const double sd = r[k], td = q[k];
                c[k] = td * sd;
                c[NR + k] = td * td;
                c[2 * NR + k] = wd * sd * sd;
            }
        } else if (step == kExit || step == kCap) {
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const double rd = rhs(k) - q[k];
                c[k] = wd * rd * rd;
            }
        } else {
            nv = step == kStart ? 3 * NR : 2 * NR;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                if (step == kStart) {
                    const T bk = rhs(k);
                    const double bd = bk;
                    r[k] = a.inner ? bk : bk - q[k];
                    set_h(k, r[k]);
                    c[2 * NR + k] = wd * bd * bd;
                } else if (step == kCheck && ((cands >> k) & 1)) {
                    r[k] = rhs(k) - q[k];
                }
                const double rd = r[k];
                c[k] = static_cast<double>(hk(k)) * rd;
                c[NR + k] = wd * rd * rd;
            }
        }
        if (!total(c, nv)) break;
        const double s0 = all[lk], tol2 = get(kTol2 + lk);
        if (step == kCap) {
            const int met = those(s0 <= tol2);
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if ((active >> k) & 1) done(k, (met >> k) & 1 ? OASIS_OK : OASIS_ENOTCONV, it, all[k]);
            break;
        }
        if (step == kP) {
            const int nan = those(!finite(s0)) & active, zero = those(s0 == 0.0) & active;
            if (nan | zero) {
                int any = 0;
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    if ((nan >> k) & 1) done(k, OASIS_ENAN, it, NAN);
                    if ((zero >> k) & 1) any |= restart(k);
                }
                if (!active) break;
                if (any) step = kNorms;           // else the step again, for those that are left
                continue;
            }
            const double rr = get(kRr + lk);
            put(kRho, rr);
            put(kAlpha, rr / s0);
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                u[k] = vec[k * LEN + t];          // p, until the next u takes its place
                r[k] = fms_t(r[k], static_cast<T>(get(kAlpha + k)), vk(k));   // s in r's place
            }
            step = kS;
            continue;
        }
        if (step == kS || step == kExit) {
            int met;
            if (step == kS) {
                met = those(all[2 * NR + lk] <= tol2) & active;
                cands = 0;
#pragma unroll
                for (int k = 0; k < NR; ++k)
                    if (((met >> k) & 1) && no_sexit[k] != it) cands |= 1 << k;
                const double tt = all[NR + lk];
                put(kOmega, tt > 0.0 ? s0 / tt : 0.0);
                if (cands && !a.inner) {
                    if (own) {
#pragma unroll
                        for (int k = 0; k < NR; ++k) {
                            item<T>(a.keep_s[k], off) = r[k];
                            item<T>(a.keep_t[k], off) = q[k];
                        }
                    }
                    step = kExit;
                    continue;
                }
            } else {
                met = those(s0 <= tol2);
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    r[k] = item<const T>(a.keep_s[k], off);
                    q[k] = item<const T>(a.keep_t[k], off);
                }
            }
            // the candidates by their explicit residuals, or (inner) the norms of s
            if (cands) {
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    if (!((cands >> k) & 1)) continue;
                    if ((met >> k) & 1) {
                        if (own) xk(k) = xk(k) + static_cast<T>(get(kAlpha + k)) * u[k];
                        done(k, OASIS_OK, it + 1, all[step == kS ? 2 * NR + k : k]);
                    } else {
                        no_sexit[k] = it;
                        again[k] += 1;
                    }
                }
                if (!active) break;
            }
            // x += alpha p + omega s, r = s - omega t, u = p - omega v
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                const T al = static_cast<T>(get(kAlpha + k)), om = static_cast<T>(get(kOmega + k));
                if (own && ((active >> k) & 1)) xk(k) = xk(k) + al * u[k] + om * r[k];
                r[k] = fms_t(r[k], om, q[k]);
                u[k] = fms_t(u[k], om, vk(k));
            }
            ++it;
            step = kNorms;
            continue;
        }
        // kStart, kCheck, kNorms: the norms of the residuals as they are
        const double wr = all[NR + lk];
        put(kRr, s0);
        double tol = tol2;
        if (step == kStart) {
            tol = a.rtol2 * all[2 * NR + lk];
            put(kTol2, tol);
            if (t < NR) result[t].wbb = all[2 * NR + t];
        }
        const int met = those(wr <= tol);
        if (step == kCheck) {
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                if (!((cands >> k) & 1)) continue;
                if ((met >> k) & 1)
                    done(k, OASIS_OK, it, all[NR + k]);
                else
                    again[k] += 1;                // the explicit residual replaces the recursive one
            }
            if (!active) break;
        }
        if (it >= a.maxit) {
            step = kCap;
            continue;
        }
        // tests of the incoming residual
        const int nan = those(!finite(s0) || !finite(wr)) & active;
        const int broken = those(s0 == 0.0 || get(kOmega + lk) == 0.0) & active & ~nan & ~met;
        cands = met & active & ~nan;
        if (nan | broken | cands) {
            int any = 0;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                if ((nan >> k) & 1) done(k, OASIS_ENAN, it, NAN);
                // inner: trusted, the caller's FP64 residual decides
                if (a.inner && ((cands >> k) & 1)) done(k, OASIS_OK, it, all[NR + k]);
            }
            if (cands && !a.inner) {
                step = kCheck;                    // those that are broken down are seen again after it
                continue;
            }
#pragma unroll
            for (int k = 0; k < NR; ++k)
                if ((broken >> k) & 1) any |= restart(k);
            if (!active) break;
            if (any) {
                step = kNorms;
                continue;
            }
        }
        put(kBeta, (s0 / get(kRho + lk)) * (get(kAlpha + lk) / get(kOmega + lk)));
        step = kP;
    }
    if (quit[0] | quit[1]) {
        // (a block that was told leaves the flag as it is)
        if (t == 0 && ((quit[0] | quit[1]) & kRanOut)) atomicMax(flag, waits == 1 ? kCoopLate : kCoopLost);
        return;
    }
    if (bid == 0 && t == 0) {
        for (int k = 0; k < NR; ++k) a.blk->st[k] = result[k];
    }
}

// the words and slots that are sent before they have been emptied: those of
// the first two vectors and sums; the start iterate and the flag
template <typename T>
__global__ __launch_bounds__(kBlock) void k_bi_coop_clear(int words, int slots, BiCoopArgs a) {
    const int step = gridDim.x * blockDim.x, i0 = blockIdx.x * blockDim.x + threadIdx.x;
    for (int k = 0; k < 2; ++k)
        for (int i = i0; i < words; i += step) static_cast<typename Word<T>::U *>(a.ex[k])[i] = Word<T>::kEmpty;
    for (int i = i0; i < slots; i += step) a.slots[i] = Word<double>::kEmpty;
    if (a.x0)
        for (int k = 0; k < words / a.n; ++k)
            for (int i = i0; i < a.n; i += step)
                static_cast<T *>(a.x0)[k * a.n + i] = static_cast<const T *>(a.x[k])[i];
    if (i0 == 0) a.blk->glob.pause = 0;
}

// x as it was at the start
template <typename T>
__global__ __launch_bounds__(kBlock) void k_bi_coop_back(int nrhs, BiCoopArgs a) {
    for (int k = 0; k < nrhs; ++k)
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += gridDim.x * blockDim.x)
            static_cast<T *>(a.x[k])[i] = static_cast<const T *>(a.x0)[k * a.n + i];
}

template <typename T, int NR>
int launch(hipStream_t s, int grid, BiCoopArgs &a) {
    void *args[] = {&a};
    const void *kern;
    int bs;
    if (a.rows <= 256) {
        kern = reinterpret_cast<const void *>(&k_bi_coop<T, NR, 256>);
        bs = 256;
    } else if (a.rows <= 512) {
        kern = reinterpret_cast<const void *>(&k_bi_coop<T, NR, 512>);
        bs = 512;
    } else {
        kern = reinterpret_cast<const void *>(&k_bi_coop<T, NR, 1024>);
        bs = 1024;
    }
    if (hipLaunchKernel(kern, dim3(grid), dim3(bs), args, 0, s) != hipSuccess) {
        (void)hipGetLastError();
        return OASIS_EUNSUPPORTED;
    }
    return OASIS_OK;
}

}  // namespace

template <typename T>
int bicg_coop_solve(hipStream_t s, int n, int nrhs, const T *wgt, const T *const *b, T *const *x, double rtol, int maxit,
                    BiWork<T> &w, SolveOut *out, bool inner, int *lost) {
    // one row per thread of one block per CU; a kernel and grid that the
    // caller asked for are left as they are.  An iteration takes 11 to 40 us:
    // kCoopRun of them bound a launch that does not converge to 0.16 s.  A
    // higher cap, the entry points' default of 10000 among them, takes the
    // launched form from the start: a solve is not handed over in the middle.
    if (!w.cols.any() || !w.eval || !w.tun.ell() || !w.tun.grid_auto || n > kCoopMaxRows ||
        maxit > kCoopRun)
        return OASIS_EUNSUPPORTED;
    int most = 0;
    OASIS_TRY(coop_blocks(s, &most));
    if (n > most * kCoopThreads || !w.coop.next()) return OASIS_EUNSUPPORTED;
    const int grid = std::min(most, (n + kBlock - 1) / kBlock);
    BiCoopArgs a{};
    a.n = n;
    a.rows = (n + grid - 1) / grid;
    a.cols = w.cols;
    a.eval = w.eval;
    a.wgt = wgt;
    for (int k = 0; k < nrhs; ++k) {
        a.b[k] = b[k];
        a.x[k] = x[k];
        a.v[k] = w.p[k];
        a.rhat[k] = w.rhat[k];
        a.keep_s[k] = w.xs[k];
        a.keep_t[k] = w.t[k];
    }
    a.blk = reinterpret_cast<BiBlock *>(w.st);
    a.rtol2 = rtol * rtol;
    a.maxit = maxit;
    a.inner = inner ? 1 : 0;
    // the words live in the (r, v) and (r, u) pairs, the start iterate too, and
    // the slots in the partial arrays, which this form does not use
    const int words = n * nrhs;
    a.ex[0] = w.rv;
    a.ex[1] = reinterpret_cast<T *>(w.rv) + words;
    a.ex[2] = w.ru;
    a.x0 = inner ? nullptr : reinterpret_cast<T *>(w.ru) + words;
    a.slots = reinterpret_cast<u64 *>(w.part1);
    // (a set: 3 nrhs values, copies, blocks; part1, part2 and part3 hold
    // three sets of 9 values of kMaxPartials = 8 copies of 256 blocks)
    constexpr int kWords = 3 * 9 * kMaxPartials;
    if (w.part3 != w.part1 + 2 * 9 * kMaxPartials) return OASIS_EUNSUPPORTED;
    a.copies = std::min(kXcds, kWords / (4 * 3 * nrhs * grid));
    BiBlock h{};
    for (int attempt = 0;; ++attempt) {
        a.join = join_ticks();
        a.lose = lose_wait(w.lose, attempt);
        hipLaunchKernelGGL(k_bi_coop_clear<T>, dim3(grid_for(words, kBlock, 1024)), dim3(kBlock), 0, s, words,
                           2 * 3 * nrhs * a.copies * grid, a);
        OASIS_TRY_LAUNCH();
        OASIS_TRY(nrhs == 1 ? (launch<T, 1>(s, grid, a)) : nrhs == 2 ? (launch<T, 2>(s, grid, a)) : (launch<T, 3>(s, grid, a)));
        OASIS_TRY(read_state(s, w.stage, a.blk, &h, sizeof(h)));
        if (h.glob.pause == 0) break;
        *lost += 1;
        if (h.glob.pause != kCoopUnfit && a.x0) {
            hipLaunchKernelGGL(k_bi_coop_back<T>, dim3(grid_for(n, kBlock, 1024)), dim3(kBlock), 0, s, nrhs, a);
            OASIS_TRY_LAUNCH();
        }
        if (h.glob.pause == kCoopUnfit) {
            w.coop.never = true;
            return OASIS_EUNSUPPORTED;
        }
        // (a wait of 2 s is not taken twice over)
        if (attempt + 1 >= (h.glob.pause == kCoopLate ? kCoopTries : 2)) {
            w.coop.gave_up();
            return OASIS_EUNSUPPORTED;
        }
    }
    w.coop.worked();
    int worst = OASIS_OK;
    for (int k = 0; k < nrhs; ++k) {
        const BiState &o = h.st[k];
        out[k] = SolveOut();
        out[k].status = o.event;
        out[k].iters = o.it_rec;
        out[k].replacements = o.active;
        out[k].coop = 1;
        out[k].lost = *lost;
        if (!(o.wrr_rec < 0.0)) out[k].rel_res = o.wbb > 0.0 ? std::sqrt(o.wrr_rec / o.wbb) : std::sqrt(o.wrr_rec);
        if (o.event != OASIS_OK && (worst == OASIS_OK || o.event < worst)) worst = o.event;
    }
    return worst;
}

template int bicg_coop_solve<double>(hipStream_t, int, int, const double *, const double *const *, double *const *,
                                     double, int, BiWork<double> &, SolveOut *, bool, int *);
template int bicg_coop_solve<float>(hipStream_t, int, int, const float *, const float *const *, float *const *, double,
                                    int, BiWork<float> &, SolveOut *, bool, int *);

}  // namespace oasis
