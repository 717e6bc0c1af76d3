// Graph set-up on the device: the shared P1 sparsity pattern, greedy cell
// colouring for atomic-free assembly, colour classes, and the reverse
// Cuthill-McKee ordering.  All results are deterministic: integer atomics
// only count or claim, and every order-dependent list is re-sorted by a
// total key before use.
#include <algorithm>
#include <cstring>
#include <vector>

#include "internal.hpp"

namespace oasis {

// ---------------------------------------------------------------------------
// exclusive scan of int32 (n <= 2^31 - 1 total), out[n] = total

constexpr int kScanTile = 1024;   // elements per block (256 threads x 4)

__global__ __launch_bounds__(kBlock) void k_scan_tiles(int n, const int *__restrict__ in,
                                                       int *__restrict__ out,
                                                       int *__restrict__ tile_sums) {
    __shared__ int sh[kScanTile];
    const int base = blockIdx.x * kScanTile;
    for (int k = threadIdx.x; k < kScanTile; k += blockDim.x)
        sh[k] = (base + k < n) ? in[base + k] : 0;
    __syncthreads();
    // each thread scans 4 consecutive elements, then a Hillis-Steele pass over thread totals
    const int t = threadIdx.x;
    int a0 = sh[4 * t], a1 = sh[4 * t + 1], a2 = sh[4 * t + 2], a3 = sh[4 * t + 3];
    int tot = a0 + a1 + a2 + a3;
    __shared__ int ts[kBlock];
    ts[t] = tot;
    __syncthreads();
    for (int o = 1; o < kBlock; o <<= 1) {
        int v = (t >= o) ? ts[t - o] : 0;
        __syncthreads();
        ts[t] += v;
        __syncthreads();
    }
    int excl = ts[t] - tot;
    sh[4 * t] = excl;
    sh[4 * t + 1] = excl + a0;
    sh[4 * t + 2] = excl + a0 + a1;
    sh[4 * t + 3] = excl + a0 + a1 + a2;
    __syncthreads();
    for (int k = threadIdx.x; k < kScanTile; k += blockDim.x)
        if (base + k < n) out[base + k] = sh[k];
    if (t == kBlock - 1) tile_sums[blockIdx.x] = ts[t];
}

// single block: exclusive scan of the tile sums in place, total at [ntiles]
__global__ __launch_bounds__(1024) void k_scan_sums(int ntiles, int *sums) {
    __shared__ int carry;
    __shared__ int ts[1024];
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < ntiles; base += 1024) {
        const int i = base + threadIdx.x;
        const int v = i < ntiles ? sums[i] : 0;
        ts[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            int a = (threadIdx.x >= (unsigned)o) ? ts[threadIdx.x - o] : 0;
            __syncthreads();
            ts[threadIdx.x] += a;
            __syncthreads();
        }
        if (i < ntiles) sums[i] = carry + ts[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == 1023) carry += ts[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[ntiles] = carry;
}

__global__ __launch_bounds__(kBlock) void k_scan_add(int n, int *out, const int *sums, int *total) {
    const int i = blockIdx.x * kScanTile;
    const int off = sums[blockIdx.x];
    for (int k = threadIdx.x; k < kScanTile; k += blockDim.x)
        if (i + k < n) out[i + k] += off;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        out[n] = sums[gridDim.x];
        if (total) *total = sums[gridDim.x];
    }
}

static size_t scan_ws_ints(int n) { return (size_t)(n + kScanTile - 1) / kScanTile + 1; }

// out has n+1 entries; in may equal out only if n == 0; total (nullable)
// receives out[n] too
static int exclusive_scan(hipStream_t s, int n, const int *in, int *out, int *tmp, int *total = nullptr) {
    const int tiles = std::max(1, (n + kScanTile - 1) / kScanTile);
    hipLaunchKernelGGL(k_scan_tiles, dim3(tiles), dim3(kBlock), 0, s, n, in, out, tmp);
    OASIS_TRY_LAUNCH();
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, s, tiles, tmp);
    OASIS_TRY_LAUNCH();
    hipLaunchKernelGGL(k_scan_add, dim3(tiles), dim3(kBlock), 0, s, n, out, tmp, total);
    OASIS_TRY_LAUNCH();
    return OASIS_OK;
}

__global__ __launch_bounds__(kBlock) void k_fill_i(long long n, int *x, int v) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        x[i] = v;
}

static int fill_i(hipStream_t s, long long n, int *x, int v) {
    if (n <= 0) return OASIS_OK;
    const int g = (int)std::min<long long>((n + kBlock - 1) / kBlock, 8192);
    hipLaunchKernelGGL(k_fill_i, dim3(g), dim3(kBlock), 0, s, n, x, v);
    OASIS_TRY_LAUNCH();
    return OASIS_OK;
}

// ---------------------------------------------------------------------------
// dof -> incident cells, stored as codes cell * (dim+1) + local vertex,
// each list ascending

__global__ __launch_bounds__(kBlock) void k_inc_count(int ncell, int nv, int nvert, int ndof,
                                                      const int *__restrict__ cells,
                                                      const int *__restrict__ v2d, int *cnt,
                                                      int *err) {
    for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < ncell;
         c += (long long)gridDim.x * blockDim.x) {
        int d[4];
        bool ok = true;
        for (int a = 0; a < nv; ++a) {
            const int v = cells[c * nv + a];
            if (v < 0 || v >= nvert) {
                ok = false;
                d[a] = -1;
                continue;
            }
            d[a] = v2d[v];
            if (d[a] < 0 || d[a] >= ndof) ok = false;
        }
        if (!ok) {
            atomicOr(err, 2);   // index out of range: the mesh is rejected
            continue;
        }
        for (int a = 0; a < nv; ++a) {
            for (int b = 0; b < a; ++b)
                if (d[a] == d[b]) atomicOr(err, 1);   // a cell must hold distinct dofs
            atomicAdd(&cnt[d[a]], 1);
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_inc_fill(int ncell, int nv, const int *__restrict__ cells,
                                                     const int *__restrict__ v2d,
                                                     const int *__restrict__ ptr, int *fillc,
                                                     int *inc, const int *err) {
    if (*err) return;   // no index of a rejected mesh is followed
    for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < ncell;
         c += (long long)gridDim.x * blockDim.x) {
        for (int a = 0; a < nv; ++a) {
            const int d = v2d[cells[c * nv + a]];
            const int slot = atomicAdd(&fillc[d], 1);
            inc[ptr[d] + slot] = (int)(c * nv + a);   // cell and local vertex
        }
    }
}

// make every incidence list ascending (removes the fill order)
__global__ __launch_bounds__(kBlock) void k_inc_sort(int ndof, const int *__restrict__ ptr, int *inc) {
    for (long long d = blockIdx.x * (long long)blockDim.x + threadIdx.x; d < ndof;
         d += (long long)gridDim.x * blockDim.x) {
        const int s = ptr[d], e = ptr[d + 1];
        for (int i = s + 1; i < e; ++i) {
            const int v = inc[i];
            int j = i - 1;
            while (j >= s && inc[j] > v) {
                inc[j + 1] = inc[j];
                --j;
            }
            inc[j + 1] = v;
        }
    }
}

// What a workspace's incidence lists are of, and what the columns' pass wants
// them to be, with the columns that there is room for.  First in the
// workspace: whatever else is put there (colour classes) writes over it.
struct ListsOf {
    int magic, dim, n_cell, n_dof, room, bad;
    static constexpr int kMagic = 0x6f617369;
};

// Distinct neighbour dofs of each dof, ascending; count only when col ==
// nullptr.  One thread per dof reads its cells once and keeps the distinct
// dofs in its column of LDS (they are few: 15 on Kuhn-split hexahedra, 7 on
// right triangles, where a dof meets 24 cells of 4 or 6 of 3); a row with
// more than kPatCap of them selects the next larger dof over and over
// instead.  Bound by the gathers incidence -> vertices -> dofs: selecting
// for every row read them once per entry, 1.60 ms per pass on 112,000 dofs
// of a randomly numbered mesh; 0.11 ms this way.
// The pass that counts (len) says in `lists` what the lists are of; the one
// that writes the columns (col) does so only if that is what it wants, and
// only the rows for which rp has the place; else lists->bad is raised.
constexpr int kPatBlock = 128, kPatCap = 32;
template <int NV>
__global__ __launch_bounds__(kPatBlock) void k_row_pattern(int ndof, const int *__restrict__ cells,
                                                           const int *__restrict__ v2d,
                                                           const int *__restrict__ iptr,
                                                           const int *__restrict__ inc,
                                                           const int *__restrict__ rp, int *len, int *col,
                                                           ListsOf want, ListsOf *lists, const int *err) {
    __shared__ int seen[kPatCap][kPatBlock];
    const int t = threadIdx.x;
    if (!col) {
        if (*err) return;
        if (blockIdx.x == 0 && t == 0) *lists = want;
    } else if (lists->magic != want.magic || lists->dim != want.dim || lists->n_cell != want.n_cell ||
               lists->n_dof != want.n_dof) {
        if (blockIdx.x == 0 && t == 0) lists->bad = 1;
        return;
    }
    // whether rp has `count` entries for row d, and the columns room for them
    auto room = [&](long long d, int count) -> bool {
        const int out = rp[d];
        if (out >= 0 && count >= 0 && rp[d + 1] - out == count && count <= want.room - out) return true;
        atomicOr(&lists->bad, 1);
        return false;
    };
    for (long long d = blockIdx.x * (long long)kPatBlock + t; d < ndof; d += (long long)gridDim.x * kPatBlock) {
        const int s = iptr[d], e = iptr[d + 1];
        int count = 0;
        for (int i = s; i < e && count <= kPatCap; i += 4) {
            int q[4][NV];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const long long c = inc[i + u < e ? i + u : i] / NV;
#pragma unroll
                for (int a = 0; a < NV; ++a) q[u][a] = v2d[cells[c * NV + a]];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int a = 0; a < NV; ++a) {
                    bool old = false;
                    for (int k = 0; k < count && k < kPatCap; ++k) old |= seen[k][t] == q[u][a];
                    if (!old) {
                        if (count < kPatCap) seen[count][t] = q[u][a];
                        ++count;
                    }
                }
        }
        if (count <= kPatCap) {
            if (col && room(d, count)) {
                const int out = rp[d];
                for (int k = 0; k < count; ++k) {
                    const int v = seen[k][t];
                    int at = 0;
                    for (int m = 0; m < count; ++m) at += seen[m][t] < v ? 1 : 0;
                    col[out + at] = v;
                }
            }
        } else {
            const int most = col ? rp[d + 1] - rp[d] : 0x7fffffff;
            if (col && !room(d, most)) continue;
            int prev = -1, out = col ? rp[d] : 0;
            count = 0;
            while (true) {
                int best = 0x7fffffff;
                for (int i = s; i < e; ++i) {
                    const long long c = inc[i] / NV;
                    for (int a = 0; a < NV; ++a) {
                        const int q = v2d[cells[c * NV + a]];
                        if (q > prev && q < best) best = q;
                    }
                }
                if (best == 0x7fffffff || count == most) {
                    if (col && (best != 0x7fffffff || count != most)) atomicOr(&lists->bad, 1);
                    break;
                }
                if (col) col[out++] = best;
                ++count;
                prev = best;
            }
        }
        if (!col) len[d] = count;
    }
}

struct GraphWs {
    ListsOf *lists;
    int *iptr, *inc, *cnt, *tmp, *flag;
    int *round_of, *color_cnt, *pos, *more;
    unsigned long long *used;
};

static void carve_graph(Carver &c, const oasis_mesh *m, GraphWs &g) {
    const long long nv = m->dim + 1;
    const int nmax = std::max(m->n_dof, m->n_cell);
    int *head = c.take<int>(32);
    g.lists = reinterpret_cast<ListsOf *>(head);
    g.flag = head ? head + 16 : nullptr;
    g.iptr = c.take<int>((size_t)m->n_dof + 1);
    g.inc = c.take<int>((size_t)m->n_cell * nv);
    g.cnt = c.take<int>((size_t)nmax + 1);
    g.tmp = c.take<int>(scan_ws_ints(nmax) + 16);
    g.round_of = c.take<int>((size_t)m->n_cell);
    g.color_cnt = c.take<int>(256);
    g.pos = c.take<int>((size_t)nmax + 1);
    g.more = c.take<int>((size_t)m->n_cell);
    g.used = c.take<unsigned long long>(2 * (size_t)m->n_dof);
}

static int check_mesh(const oasis_mesh *m) {
    if (!m || (m->dim != 2 && m->dim != 3) || m->n_vert <= 0 || m->n_cell <= 0 || m->n_dof <= 0)
        return OASIS_EINVAL;
    if (!m->coords || !m->cells || !m->vert2dof) return OASIS_EINVAL;
    return OASIS_OK;
}

// what g.flag[0] says of a mesh (k_inc_count)
static int mesh_status(int err) {
    return err == 0 ? OASIS_OK : err & 2 ? OASIS_EINVAL : OASIS_EUNSUPPORTED;
}

// sorted: every list ascending (the pattern and the colouring do not depend
// on the order within a list).  Not `look`: the caller reads g.flag itself,
// and until then no kernel may follow the lists where it is not zero.
static int build_incidence(hipStream_t s, const oasis_mesh *m, GraphWs &g, bool sorted, bool look = true) {
    const int nv = m->dim + 1;
    const int gc = grid_for(m->n_cell, kBlock, 8192);
    OASIS_TRY(fill_i(s, m->n_dof + 1, g.cnt, 0));
    if (g.lists)   // (and the flags behind it)
        OASIS_TRY(fill_i(s, 32, &g.lists->magic, 0));
    else
        OASIS_TRY(fill_i(s, 16, g.flag, 0));
    hipLaunchKernelGGL(k_inc_count, dim3(gc), dim3(kBlock), 0, s, m->n_cell, nv, m->n_vert, m->n_dof,
                       m->cells, m->vert2dof, g.cnt, g.flag);
    OASIS_TRY_LAUNCH();
    if (look) {
        int err = 0;
        OASIS_TRY_HIP(hipMemcpyAsync(&err, g.flag, sizeof(int), hipMemcpyDeviceToHost, s));
        OASIS_TRY_HIP(hipStreamSynchronize(s));
        OASIS_TRY(mesh_status(err));
    }
    OASIS_TRY(exclusive_scan(s, m->n_dof, g.cnt, g.iptr, g.tmp));
    OASIS_TRY(fill_i(s, m->n_dof + 1, g.cnt, 0));
    hipLaunchKernelGGL(k_inc_fill, dim3(gc), dim3(kBlock), 0, s, m->n_cell, nv, m->cells,
                       m->vert2dof, g.iptr, g.cnt, g.inc, g.flag);
    OASIS_TRY_LAUNCH();
    if (sorted) {
        hipLaunchKernelGGL(k_inc_sort, dim3(grid_for(m->n_dof, kBlock, 8192)), dim3(kBlock), 0, s, m->n_dof, g.iptr,
                           g.inc);
        OASIS_TRY_LAUNCH();
    }
    return OASIS_OK;
}

// Incidence lists for an external user (the IPCS handle): iptr [n_dof+1],
// inc [n_cell*(dim+1)], scratch cnt [max(n_dof, n_cell)+1], tmp (scan).
int incidence_codes(hipStream_t s, const oasis_mesh *m, int *iptr, int *inc, int *cnt, int *tmp, int *flag) {
    GraphWs g{};
    g.iptr = iptr;
    g.inc = inc;
    g.cnt = cnt;
    g.tmp = tmp;
    g.flag = flag;
    return build_incidence(s, m, g, true);
}

size_t incidence_tmp_ints(int n) { return scan_ws_ints(n) + 16; }

// ---------------------------------------------------------------------------
// A block's appends to a global list: collected in LDS and placed with one
// atomic on the list's size (with one per append a round took 49 us, with
// one per block 19).  All threads construct and flush; push is for any thread.
constexpr int kQueueCap = 2048;
struct BlockQueue {
    int *buf, *n, *out, *size;
    __device__ __forceinline__ BlockQueue(int *lds, int *out_, int *size_)
        : buf(lds + 2), n(lds), out(out_), size(size_) {
        if (threadIdx.x == 0) *n = 0;
        __syncthreads();
    }
    __device__ __forceinline__ void push(int v) {
        const int i = atomicAdd(n, 1);
        if (i < kQueueCap)
            buf[i] = v;
        else
            out[atomicAdd(size, 1)] = v;
    }
    __device__ __forceinline__ void flush() {
        __syncthreads();
        const int m = min(*n, kQueueCap);
        if (m == 0) return;
        if (threadIdx.x == 0) n[1] = atomicAdd(size, m);
        __syncthreads();
        const int at = n[1];
        for (int i = threadIdx.x; i < m; i += blockDim.x) out[at + i] = buf[i];
    }
};

// ---------------------------------------------------------------------------
// greedy first-fit colouring in decreasing priority
//
// Every dof has its cells in decreasing priority and points at the first one
// without a colour.  A cell whose turn it is at all its dofs has no uncoloured
// neighbour of higher priority: it takes the first colour that none of its
// dofs has seen, marks it there, and moves the pointers on, which may make it
// some other cell's turn in the next round.  That is 12 accesses and 4 atomics
// a cell, where counting each cell's neighbours and notifying them one by one
// took 100 of each: on 618,000 randomly numbered cells 160 rounds of 17 us
// and 0.37 ms for the first count, now 6.9 us and 0.14 ms for the sort.  A
// round is a chain of seven dependent accesses.  (Blocks that colour what they
// made ready themselves, without a launch in between, run out of cells while
// a few have all of them: 35 us a step.)
constexpr int kColorList = 128;   // the cells of a dof have colours of their own, at most 128

// The cells of every dof in decreasing priority, in place of their codes; the
// first one's turn.  A wave a dof.  Bits of *bad: 1 too many cells for 128
// colours, 2 equal priorities.
template <int NV>
__global__ __launch_bounds__(kBlock) void k_color_sort(int ndof, const int *__restrict__ iptr, int *inc,
                                                       const int *__restrict__ pri, int *head,
                                                       unsigned long long *used, int *turns, int *queue, int *size,
                                                       int *bad) {
    constexpr int WAVES = kBlock / kWave;
    __shared__ int lds[kQueueCap + 2];
    __shared__ int cell[WAVES][kColorList], key[WAVES][kColorList];
    BlockQueue ready(lds, queue, size);
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    for (int d = blockIdx.x * WAVES + wv; d < ndof; d += gridDim.x * WAVES) {
        const int b = iptr[d], n = iptr[d + 1] - b;
        if (lane == 0) {
            head[d] = b;
            used[2 * d] = used[2 * d + 1] = 0ull;
            if (n > kColorList) atomicOr(bad, 1);
        }
        if (n > kColorList) continue;
        for (int i = lane; i < n; i += kWave) {
            const int c = inc[b + i] / NV;
            cell[wv][i] = c;
            key[wv][i] = pri[c];
        }
        wave_lds_sync();
        for (int i = lane; i < n; i += kWave) {
            const int c = cell[wv][i], p = key[wv][i];
            int r = 0;
            bool tie = false;
            for (int q = 0; q < n; ++q) {
                const int pq = key[wv][q];
                r += pq > p || (pq == p && q < i) ? 1 : 0;
                tie |= pq == p && q != i;
            }
            inc[b + r] = c;
            if (tie) atomicOr(bad, 2);
            if (r == 0 && atomicAdd(&turns[c], 1) + 1 == NV) ready.push(c);
        }
        wave_lds_sync();
    }
    ready.flush();
}

// colours the size[0] cells of queue; next / size[1]: the round after.  Four
// lanes a cell, one a vertex.
template <int NV>
__global__ __launch_bounds__(kBlock) void k_color_round(const int *__restrict__ cells, const int *__restrict__ v2d,
                                                        const int *__restrict__ iptr, const int *__restrict__ list,
                                                        int *head, unsigned long long *used, int *turns, int *color,
                                                        const int *__restrict__ queue, int *next, int *size,
                                                        int *bad) {
    constexpr int QUADS = kBlock / 4;
    __shared__ int lds[kQueueCap + 2];
    const int m = size[0];
    const int a = threadIdx.x & 3;
    const long long q0 = static_cast<long long>(blockIdx.x) * QUADS;
    if (q0 >= m) return;
    BlockQueue ready(lds, next, size + 1);
    for (long long q = q0 + threadIdx.x / 4; q < m; q += static_cast<long long>(gridDim.x) * QUADS) {
        const int c = queue[q];
        unsigned long long u0 = 0ull, u1 = 0ull;
        int d = 0, at = 0, e = 0;
        if (a < NV) {
            d = v2d[cells[static_cast<long long>(c) * NV + a]];
            u0 = used[2 * static_cast<long long>(d)];
            u1 = used[2 * static_cast<long long>(d) + 1];
            at = head[d] + 1;
            e = iptr[d + 1];
        }
        unsigned long long s0 = u0, s1 = u1;
        for (int o = 2; o > 0; o >>= 1) {
            s0 |= __shfl_xor(s0, o, 4);
            s1 |= __shfl_xor(s1, o, 4);
        }
        int k = 127;
        if (~s0)
            k = __builtin_ctzll(~s0);
        else if (~s1)
            k = 64 + __builtin_ctzll(~s1);
        else if (a == 0)
            atomicOr(bad, 1);
        if (a == 0) color[c] = k;
        if (a >= NV) continue;
        // no other cell of this round is on this dof
        if (k < 64)
            used[2 * static_cast<long long>(d)] = u0 | 1ull << k;
        else
            used[2 * static_cast<long long>(d) + 1] = u1 | 1ull << (k - 64);
        head[d] = at;
        if (at == e) continue;
        const int nx = list[at];
        if (atomicAdd(&turns[nx], 1) + 1 == NV) ready.push(nx);
    }
    ready.flush();
}

// the sizes of a batch of rounds: the last becomes the first, the rest zero
__global__ __launch_bounds__(kBlock) void k_color_carry(int rounds, int *size) {
    const int last = size[rounds];
    __syncthreads();
    for (int i = threadIdx.x; i <= rounds; i += blockDim.x) size[i] = i == 0 ? last : 0;
}

__global__ __launch_bounds__(kBlock) void k_color_count(int ncell, const int *color, int *cnt) {
    __shared__ int h[128];
    for (int i = threadIdx.x; i < 128; i += blockDim.x) h[i] = 0;
    __syncthreads();
    for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < ncell;
         c += (long long)gridDim.x * blockDim.x)
        atomicAdd(&h[color[c]], 1);
    __syncthreads();
    for (int i = threadIdx.x; i < 128; i += blockDim.x)
        if (h[i]) atomicAdd(&cnt[i], h[i]);
}

// Colour classes as a stable counting sort over tiles of kBlock cells.
// k_class_count: cells of each colour in each tile, at hist[colour * tiles +
// tile] (their exclusive scan gives every tile's first place in a class);
// k_class_fill: each cell's place, from the waves' counts and the cell's rank
// among the equal colours of its wave.  Colours outside [0, n_colors) are
// left out.
constexpr int kClassWaves = kBlock / kWave;

// lanes of the wave whose colour equals this lane's (0 when it has none)
__device__ __forceinline__ unsigned long long same_color(int k, bool in) {
    unsigned long long m = __ballot(in);
#pragma unroll
    for (int b = 0; b < 7; ++b) {
        const unsigned long long w = __ballot((k >> b) & 1);
        m &= (k >> b) & 1 ? w : ~w;
    }
    return in ? m : 0ull;
}

__global__ __launch_bounds__(kBlock) void k_class_count(int ncell, int ncol, int tiles, const int *__restrict__ color,
                                                        int *__restrict__ hist) {
    __shared__ int h[128];
    for (int i = threadIdx.x; i < 128; i += kBlock) h[i] = 0;
    __syncthreads();
    const long long c = blockIdx.x * (long long)kBlock + threadIdx.x;
    const int k = c < ncell ? color[c] : -1;
    if (k >= 0 && k < ncol) atomicAdd(&h[k], 1);
    __syncthreads();
    for (int i = threadIdx.x; i < ncol; i += kBlock) hist[(long long)i * tiles + blockIdx.x] = h[i];
}

__global__ __launch_bounds__(kBlock) void k_class_fill(int ncell, int ncol, int tiles, const int *__restrict__ color,
                                                       const int *__restrict__ first, int *__restrict__ out) {
    __shared__ int h[kClassWaves][128];
    const int wv = threadIdx.x / kWave, wl = threadIdx.x & (kWave - 1);
    for (int i = threadIdx.x; i < kClassWaves * 128; i += kBlock) h[i / 128][i & 127] = 0;
    __syncthreads();
    const long long c = blockIdx.x * (long long)kBlock + threadIdx.x;
    const int k = c < ncell ? color[c] : -1;
    const bool in = k >= 0 && k < ncol;
    const unsigned long long same = same_color(in ? k : 0, in);
    const int rank = __popcll(same & ((1ull << wl) - 1ull));
    if (in && rank == 0) h[wv][k] = __popcll(same);
    __syncthreads();
    if (!in) return;
    int at = first[(long long)k * tiles + blockIdx.x] + rank;
    for (int w = 0; w < wv; ++w) at += h[w][k];
    out[at] = static_cast<int>(c);
}

// class starts: ptr[k] = first[k * tiles], ptr[ncol] = the total
__global__ __launch_bounds__(kBlock) void k_class_ptr(int ncol, int tiles, const int *__restrict__ first, int *ptr) {
    for (int k = threadIdx.x; k <= ncol; k += blockDim.x) ptr[k] = first[(long long)k * tiles];
}

// ---------------------------------------------------------------------------
// reverse Cuthill-McKee

//
// The levels of the breadth-first passes are small and many (about 50 of
// 2,000 dofs on a 112,000-dof mesh, three to four passes), so reading each
// level's size back to launch the next cost more than the levels (25 us a
// level then, 6 in a batch).  Sizes and
// offsets of a batch of levels stay on the device: a level's kernels read
// them there, from grids that do not depend on them, and the host looks
// once per batch.

constexpr int kLevels = 16;                 // levels per batch at most
// first vertex and size of each level of a batch (and of the one after)
struct RcmLevels {
    int off[kLevels + 2], cnt[kLevels + 2];
};

struct RcmWs {
    int *pos, *dist, *claim, *lst[2], *grp, *cnt, *off, *fillc;
    RcmLevels *lev;
    long long *keyp;
};

static void carve_rcm(Carver &c, int n, RcmWs &r) {
    r.pos = c.take<int>(n);
    r.dist = c.take<int>(n);
    r.claim = c.take<int>(n);
    r.lst[0] = c.take<int>(n);
    r.lst[1] = c.take<int>(n);
    r.grp = c.take<int>(n);
    r.cnt = c.take<int>((size_t)n + 1);
    r.off = c.take<int>((size_t)n + 1);
    r.fillc = c.take<int>((size_t)n + 1);
    r.lev = c.take<RcmLevels>(1);
    r.keyp = c.take<long long>(kMaxPartials + 16);
}

__device__ __forceinline__ long long deg_key(const int *rp, int v) {
    return ((long long)(rp[v + 1] - rp[v]) << 32) | (unsigned)v;
}

// minimum (degree, index) over list[0..m) (or over unplaced vertices 0..n if list == nullptr)
__global__ __launch_bounds__(kBlock) void k_minkey(int m, const int *list, const int *rp,
                                                   const int *pos, long long *part) {
    __shared__ long long sh[kBlock];
    long long best = 0x7fffffffffffffffll;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < m;
         i += (long long)gridDim.x * blockDim.x) {
        const int v = list ? list[i] : (int)i;
        if (!list && pos[v] >= 0) continue;
        const long long k = deg_key(rp, v);
        best = k < best ? k : best;
    }
    sh[threadIdx.x] = best;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o && sh[threadIdx.x + o] < sh[threadIdx.x]) sh[threadIdx.x] = sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(kBlock) void k_minkey_final(int np, long long *part) {
    __shared__ long long sh[kBlock];
    long long best = 0x7fffffffffffffffll;
    for (int i = threadIdx.x; i < np; i += blockDim.x) best = part[i] < best ? part[i] : best;
    sh[threadIdx.x] = best;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o && sh[threadIdx.x + o] < sh[threadIdx.x]) sh[threadIdx.x] = sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[kMaxPartials] = sh[0];
}

constexpr int kBfsLanes = 8;                // lanes per vertex of a level

// the root starts level 0 of a pass: its mark, its place in the sequence
// (and its position, when it is being placed)
__global__ void k_level_root(int root, int at, int *mark, int *seq, int *pos, RcmLevels *lev) {
    mark[root] = 0;
    seq[at] = root;
    if (pos) pos[root] = at;
    for (int j = 0; j < kLevels + 2; ++j) lev->cnt[j] = j == 0 ? 1 : 0;
    lev->off[0] = at;
}

// the level after a batch of `levels` becomes its first
__global__ void k_level_carry(int levels, RcmLevels *lev) {
    const int off = lev->off[levels], cnt = lev->cnt[levels];
    for (int j = 0; j < kLevels + 2; ++j) lev->cnt[j] = j == 0 ? cnt : 0;
    lev->off[0] = off;
}

// BFS expansion of level j over not-yet-placed vertices: claim with a CAS
// and append to next (the sequence itself when next is null)
__global__ __launch_bounds__(kBlock) void k_bfs_expand(int j, const int *seq, const int *rp, const int *ci,
                                                       const int *pos, int *mark, int *seqw, int *next,
                                                       int *zero0, int *zero1, RcmLevels *lev) {
    const int b = lev->off[j], m = lev->cnt[j];
    if (blockIdx.x == 0 && threadIdx.x == 0) lev->off[j + 1] = b + m;
    const int lane = threadIdx.x & (kBfsLanes - 1);
    const int step = gridDim.x * kBlock;
    const int t0 = blockIdx.x * kBlock + threadIdx.x;
    if (zero0)
        for (int i = t0; i < m; i += step) zero0[i] = zero1[i] = 0;
    __shared__ int lds[kQueueCap + 2];
    if (blockIdx.x * (kBlock / kBfsLanes) >= m) return;
    BlockQueue found(lds, next ? next : seqw + b + m, &lev->cnt[j + 1]);
    for (int i = t0 / kBfsLanes; i < m; i += step / kBfsLanes) {
        const int u = seq[b + i];
        const int e = rp[u + 1];
        for (int k = rp[u] + lane; k < e; k += kBfsLanes) {
            const int v = ci[k];
            if (v == u || pos[v] >= 0) continue;
            if (__atomic_load_n(&mark[v], __ATOMIC_RELAXED) == -1 && atomicCAS(&mark[v], -1, 1) == -1)
                found.push(v);
        }
    }
    found.flush();
}

// parent position (least position of a placed neighbour) of the new vertices
// of level j and the child counts of level j
__global__ __launch_bounds__(kBlock) void k_cm_parent(int j, const RcmLevels *lev, const int *lst, const int *rp,
                                                      const int *ci, const int *pos, int *par, int *cnt) {
    const int lb = lev->off[j], lm = lev->cnt[j], m = lev->cnt[j + 1];
    const int lane = threadIdx.x & (kBfsLanes - 1);
    for (int i = (blockIdx.x * kBlock + threadIdx.x) / kBfsLanes; i < m; i += gridDim.x * (kBlock / kBfsLanes)) {
        const int v = lst[i], e = rp[v + 1];
        int best = 0x7fffffff;
        for (int k = rp[v] + lane; k < e; k += kBfsLanes) {
            const int p = pos[ci[k]];
            if (p >= 0 && p < best) best = p;
        }
        for (int o = kBfsLanes / 2; o > 0; o >>= 1) best = min(best, __shfl_xor(best, o, kBfsLanes));
        // with a symmetric pattern the parent lies in the previous level; clamp otherwise
        if (best < lb || best >= lb + lm) best = lb;
        if (lane == 0) {
            par[i] = best;
            atomicAdd(&cnt[best - lb], 1);
        }
    }
}

// off[p] = children of level j's vertices before p (one block)
__global__ __launch_bounds__(1024) void k_cm_offsets(int j, const RcmLevels *lev, const int *cnt, int *off) {
    constexpr int NW = 1024 / kWave;
    __shared__ int ws[NW];
    const int m = lev->cnt[j], wv = threadIdx.x / kWave, wl = threadIdx.x & (kWave - 1);
    int carry = 0;
    for (int base = 0; base < m; base += 1024) {
        const int i = base + threadIdx.x;
        const int v = i < m ? cnt[i] : 0;
        int inc = v;
        for (int o = 1; o < kWave; o <<= 1) {
            const int up = __shfl_up(inc, o, kWave);
            if (wl >= o) inc += up;
        }
        if (wl == kWave - 1) ws[wv] = inc;
        __syncthreads();
        int before = 0, all = 0;
        for (int w = 0; w < NW; ++w) {
            if (w < wv) before += ws[w];
            all += ws[w];
        }
        if (i < m) off[i] = carry + before + inc - v;
        carry += all;
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void k_cm_group(int j, const RcmLevels *lev, const int *lst, const int *par,
                                                     const int *off, int *fillc, int *grp) {
    const int lb = lev->off[j], m = lev->cnt[j + 1];
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < m; i += gridDim.x * kBlock) {
        const int p = par[i] - lb;
        const int slot = atomicAdd(&fillc[p], 1);
        grp[off[p] + slot] = lst[i];
    }
}

// siblings (same parent) are ordered by (degree, index)
__global__ __launch_bounds__(kBlock) void k_cm_place(int j, const RcmLevels *lev, const int *lst, const int *par,
                                                     const int *off, const int *cnt, const int *grp, const int *rp,
                                                     int *pos, int *order) {
    const int lb = lev->off[j], base = lb + lev->cnt[j], m = lev->cnt[j + 1];
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < m; i += gridDim.x * kBlock) {
        const int v = lst[i];
        const int p = par[i] - lb;
        const long long kv = deg_key(rp, v);
        int rank = 0;
        for (int k = off[p]; k < off[p] + cnt[p]; ++k)
            if (deg_key(rp, grp[k]) < kv) ++rank;
        const int at = base + off[p] + rank;
        pos[v] = at;
        order[at] = v;
    }
}

__global__ __launch_bounds__(kBlock) void k_rcm_finish(int n, const int *pos, const int *cm,
                                                       int *perm, int *order) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        perm[i] = n - 1 - pos[i];
        order[i] = cm[n - 1 - i];
    }
}

__global__ __launch_bounds__(kBlock) void k_relabel(int count, const int *in, const int *perm, int *out) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count;
         i += (long long)gridDim.x * blockDim.x)
        out[i] = perm[in[i]];
}

}  // namespace oasis

using namespace oasis;

// ---------------------------------------------------------------------------
// C ABI

extern "C" int oasis_graph_workspace_size(const oasis_mesh *mesh, size_t *bytes) {
    if (!bytes) return OASIS_EINVAL;
    OASIS_TRY(check_mesh(mesh));
    Carver c(nullptr, 0);
    GraphWs g;
    carve_graph(c, mesh, g);
    *bytes = c.bytes();
    return OASIS_OK;
}

// row lengths (len), or with the row offsets rp the columns into room for
// col_capacity of them, from the incidence lists in g
static int pattern_rows(hipStream_t s, const oasis_mesh *mesh, const GraphWs &g, const int *rp, int *len, int *col,
                        int64_t col_capacity) {
    const int gd = grid_for(mesh->n_dof, kPatBlock, 1 << 20);
    const ListsOf want{ListsOf::kMagic, mesh->dim, mesh->n_cell, mesh->n_dof,
                       static_cast<int>(std::min<int64_t>(col_capacity, 0x7fffffff)), 0};
    if (mesh->dim == 3)
        hipLaunchKernelGGL(k_row_pattern<4>, dim3(gd), dim3(kPatBlock), 0, s, mesh->n_dof, mesh->cells,
                           mesh->vert2dof, g.iptr, g.inc, rp, len, col, want, g.lists, g.flag);
    else
        hipLaunchKernelGGL(k_row_pattern<3>, dim3(gd), dim3(kPatBlock), 0, s, mesh->n_dof, mesh->cells,
                           mesh->vert2dof, g.iptr, g.inc, rp, len, col, want, g.lists, g.flag);
    OASIS_TRY_LAUNCH();
    return OASIS_OK;
}

// the columns; EINVAL when the lists, row_ptr or the room do not allow them
static int pattern_columns(hipStream_t s, const oasis_mesh *mesh, const GraphWs &g, const int *row_ptr, int *col_idx,
                           int64_t col_capacity) {
    OASIS_TRY(pattern_rows(s, mesh, g, row_ptr, nullptr, col_idx, col_capacity));
    int bad = 0;
    OASIS_TRY_HIP(hipMemcpyAsync(&bad, &g.lists->bad, sizeof(int), hipMemcpyDeviceToHost, s));
    OASIS_TRY_HIP(hipStreamSynchronize(s));
    if (!bad) return OASIS_OK;
    OASIS_TRY(fill_i(s, 1, &g.lists->bad, 0));   // the lists are as they were
    OASIS_TRY_HIP(hipStreamSynchronize(s));
    return OASIS_EINVAL;
}

extern "C" int oasis_p1_pattern(void *stream, const oasis_mesh *mesh, int32_t *row_ptr,
                                int32_t *col_idx, int64_t col_capacity, int32_t *nnz_out,
                                void *ws, size_t ws_bytes) {
    OASIS_TRY(check_mesh(mesh));
    if (!row_ptr || !nnz_out || !ws) return OASIS_EINVAL;
    hipStream_t s = as_stream(stream);
    Carver c(ws, ws_bytes);
    GraphWs g;
    carve_graph(c, mesh, g);
    if (!c.ok) return OASIS_EWORKSPACE;
    OASIS_TRY(build_incidence(s, mesh, g, false, false));
    OASIS_TRY(pattern_rows(s, mesh, g, nullptr, g.cnt, nullptr, 0));
    OASIS_TRY(exclusive_scan(s, mesh->n_dof, g.cnt, row_ptr, g.tmp, g.flag + 1));
    int got[2];                               // what was wrong, the entries
    OASIS_TRY_HIP(hipMemcpyAsync(got, g.flag, sizeof(got), hipMemcpyDeviceToHost, s));
    OASIS_TRY_HIP(hipStreamSynchronize(s));
    OASIS_TRY(mesh_status(got[0]));
    const int nnz = *nnz_out = got[1];
    if (!col_idx) return OASIS_OK;
    if (col_capacity < nnz) return OASIS_EINVAL;
    return pattern_columns(s, mesh, g, row_ptr, col_idx, col_capacity);
}

extern "C" int oasis_p1_pattern_columns(void *stream, const oasis_mesh *mesh, const int32_t *row_ptr,
                                        int32_t *col_idx, int64_t col_capacity, void *ws, size_t ws_bytes) {
    OASIS_TRY(check_mesh(mesh));
    if (!row_ptr || !col_idx || col_capacity < 0 || !ws) return OASIS_EINVAL;
    hipStream_t s = as_stream(stream);
    Carver c(ws, ws_bytes);
    GraphWs g;
    carve_graph(c, mesh, g);
    if (!c.ok) return OASIS_EWORKSPACE;
    return pattern_columns(s, mesh, g, row_ptr, col_idx, col_capacity);
}

extern "C" int oasis_color_cells(void *stream, const oasis_mesh *mesh, const int32_t *priority,
                                 int32_t *color, int32_t *n_colors_out, void *ws, size_t ws_bytes) {
    OASIS_TRY(check_mesh(mesh));
    if (!priority || !color || !n_colors_out || !ws) return OASIS_EINVAL;
    hipStream_t s = as_stream(stream);
    Carver c(ws, ws_bytes);
    GraphWs g;
    carve_graph(c, mesh, g);
    if (!c.ok) return OASIS_EWORKSPACE;
    OASIS_TRY(build_incidence(s, mesh, g, false));
    const int gc = grid_for(mesh->n_cell, kBlock, 8192);
    // lists of ready cells of the even and odd rounds, and the sizes of a batch
    // of rounds; the host looks once per batch
    constexpr int kRounds = 32;
    int *queue[2] = {g.round_of, g.more}, *head = g.pos, *turns = g.cnt, *size = g.color_cnt, *bad = g.flag;
    OASIS_TRY(fill_i(s, kRounds + 1, size, 0));
    OASIS_TRY(fill_i(s, 1, bad, 0));
    OASIS_TRY(fill_i(s, mesh->n_cell, turns, 0));
    const bool tet = mesh->dim == 3;
    const int gs = grid_for((long long)mesh->n_dof * kWave, kBlock, 1 << 20);
    const auto sort = tet ? k_color_sort<4> : k_color_sort<3>;
    hipLaunchKernelGGL(sort, dim3(gs), dim3(kBlock), 0, s, mesh->n_dof, g.iptr, g.inc, priority, head, g.used, turns,
                       queue[0], size, bad);
    OASIS_TRY_LAUNCH();
    const auto round = tet ? k_color_round<4> : k_color_round<3>;
    const int gr = std::min(grid_for((long long)mesh->n_cell * 4, kBlock, 1 << 20), 1024);
    int done = 0;
    while (done < mesh->n_cell) {
        for (int r = 0; r < kRounds; ++r) {
            hipLaunchKernelGGL(round, dim3(gr), dim3(kBlock), 0, s, mesh->cells, mesh->vert2dof, g.iptr, g.inc, head,
                               g.used, turns, color, queue[r & 1], queue[(r + 1) & 1], size + r, bad);
            OASIS_TRY_LAUNCH();
        }
        int h[kRounds + 1], over = 0;
        OASIS_TRY_HIP(hipMemcpyAsync(h, size, sizeof(h), hipMemcpyDeviceToHost, s));
        OASIS_TRY_HIP(hipMemcpyAsync(&over, bad, sizeof(int), hipMemcpyDeviceToHost, s));
        hipLaunchKernelGGL(k_color_carry, dim3(1), dim3(kBlock), 0, s, kRounds, size);
        OASIS_TRY_LAUNCH();
        OASIS_TRY_HIP(hipStreamSynchronize(s));
        if (over) return OASIS_EUNSUPPORTED;   // more than 128 colours, or priorities that are not distinct
        int now = 0;
        for (int r = 0; r < kRounds; ++r) now += h[r];
        done += now;
        if (now == 0 && h[kRounds] == 0 && done < mesh->n_cell) return OASIS_EUNSUPPORTED;
    }
    // number of colours = 1 + max colour
    OASIS_TRY(fill_i(s, 256, g.color_cnt, 0));
    hipLaunchKernelGGL(k_color_count, dim3(gc), dim3(kBlock), 0, s, mesh->n_cell, color, g.color_cnt);
    OASIS_TRY_LAUNCH();
    int cnt[128];
    OASIS_TRY_HIP(hipMemcpyAsync(cnt, g.color_cnt, sizeof(cnt), hipMemcpyDeviceToHost, s));
    OASIS_TRY_HIP(hipStreamSynchronize(s));
    int nc = 0;
    for (int k = 0; k < 128; ++k)
        if (cnt[k]) nc = k + 1;
    *n_colors_out = nc;
    return OASIS_OK;
}

extern "C" int oasis_color_classes(void *stream, int32_t n_cell, const int32_t *color,
                                   int32_t n_colors, int32_t *color_ptr, int32_t *color_cells,
                                   void *ws, size_t ws_bytes) {
    if (n_cell <= 0 || n_colors <= 0 || n_colors > 128 || !color || !color_ptr || !color_cells || !ws)
        return OASIS_EINVAL;
    hipStream_t s = as_stream(stream);
    Carver c(ws, ws_bytes);
    const int tiles = (n_cell + kBlock - 1) / kBlock;
    const int entries = tiles * n_colors;              // at most n_cell / 2 + 128
    int *hist = c.take<int>((size_t)entries);
    int *first = c.take<int>((size_t)entries + 1);
    int *tmp = c.take<int>(scan_ws_ints(entries) + 16);
    int *ptr = c.take<int>((size_t)n_colors + 1);
    if (!c.ok) return OASIS_EWORKSPACE;
    hipLaunchKernelGGL(k_class_count, dim3(tiles), dim3(kBlock), 0, s, n_cell, n_colors, tiles, color, hist);
    OASIS_TRY_LAUNCH();
    OASIS_TRY(exclusive_scan(s, entries, hist, first, tmp));
    hipLaunchKernelGGL(k_class_fill, dim3(tiles), dim3(kBlock), 0, s, n_cell, n_colors, tiles, color, first,
                       color_cells);
    OASIS_TRY_LAUNCH();
    hipLaunchKernelGGL(k_class_ptr, dim3(1), dim3(kBlock), 0, s, n_colors, tiles, first, ptr);
    OASIS_TRY_LAUNCH();
    OASIS_TRY_HIP(hipMemcpyAsync(color_ptr, ptr, ((size_t)n_colors + 1) * sizeof(int), hipMemcpyDeviceToHost, s));
    OASIS_TRY_HIP(hipStreamSynchronize(s));
    const int base = color_ptr[n_colors];
    return base == n_cell ? OASIS_OK : OASIS_EINVAL;
}

extern "C" int oasis_rcm_workspace_size(int32_t n, size_t *bytes) {
    if (n <= 0 || !bytes) return OASIS_EINVAL;
    Carver c(nullptr, 0);
    RcmWs r;
    carve_rcm(c, n, r);
    *bytes = c.bytes();
    return OASIS_OK;
}

static int rcm_minkey(hipStream_t s, int m, const int *list, const int *rp, const int *pos,
                      long long *part, long long *out) {
    const int g = grid_for(m, kBlock);
    hipLaunchKernelGGL(k_minkey, dim3(g), dim3(kBlock), 0, s, m, list, rp, pos, part);
    OASIS_TRY_LAUNCH();
    hipLaunchKernelGGL(k_minkey_final, dim3(1), dim3(kBlock), 0, s, g, part);
    OASIS_TRY_LAUNCH();
    OASIS_TRY_HIP(hipMemcpyAsync(out, part + kMaxPartials, sizeof(long long), hipMemcpyDeviceToHost, s));
    OASIS_TRY_HIP(hipStreamSynchronize(s));
    return OASIS_OK;
}

constexpr int kLevelGrid = 256;             // blocks of a level's kernels

// Runs `level(j)`, the launches of level j of a batch, batch by batch until
// a level is empty.  last: first vertex and size of the last level that is
// not, depth: its number.  *batch: levels to launch before the first look, and
// on return those that this pass took, which is what the next pass of the
// component takes, and the next component of a mesh in pieces of a kind (200
// triangles of their own took 121 ms in batches of 16, 36 this way; looking
// after each level they took 58).
template <class Level>
static int rcm_batches(hipStream_t s, RcmWs &r, Level level, int *batch, int *depth, int *first, int *size) {
    for (int done = 0, m = *batch;; done += m, m = std::min(2 * m, kLevels)) {
        for (int j = 0; j < m; ++j) OASIS_TRY(level(j));
        RcmLevels h;
        OASIS_TRY_HIP(hipMemcpyAsync(&h, r.lev, sizeof(h), hipMemcpyDeviceToHost, s));
        hipLaunchKernelGGL(k_level_carry, dim3(1), dim3(1), 0, s, m, r.lev);
        OASIS_TRY_LAUNCH();
        OASIS_TRY_HIP(hipStreamSynchronize(s));
        int j = 0;
        while (j < m && h.cnt[j + 1] > 0) ++j;
        if (j == m) continue;
        *depth = done + j;
        *first = h.off[j];
        *size = h.cnt[j];
        *batch = std::min(*depth + 1, kLevels);
        return OASIS_OK;
    }
}

// BFS over unplaced vertices from root; returns depth and the least-key vertex of the last level
static int rcm_levels(hipStream_t s, int n, const int *rp, const int *ci, RcmWs &r, int root, int *batch,
                      int *depth, int *last_min) {
    OASIS_TRY(fill_i(s, n, r.dist, -1));
    int *seq = r.lst[0];
    hipLaunchKernelGGL(k_level_root, dim3(1), dim3(1), 0, s, root, 0, r.dist, seq, static_cast<int *>(nullptr), r.lev);
    OASIS_TRY_LAUNCH();
    int first = 0, size = 0;
    auto level = [&](int j) -> int {
        hipLaunchKernelGGL(k_bfs_expand, dim3(kLevelGrid), dim3(kBlock), 0, s, j, seq, rp, ci, r.pos, r.dist, seq,
                           static_cast<int *>(nullptr), static_cast<int *>(nullptr), static_cast<int *>(nullptr),
                           r.lev);
        OASIS_TRY_LAUNCH();
        return OASIS_OK;
    };
    OASIS_TRY(rcm_batches(s, r, level, batch, depth, &first, &size));
    long long key = 0;
    OASIS_TRY(rcm_minkey(s, size, seq + first, rp, r.pos, r.keyp, &key));
    *last_min = (int)(key & 0xffffffffll);
    return OASIS_OK;
}

extern "C" int oasis_rcm(void *stream, int32_t n, const int32_t *row_ptr, const int32_t *col_idx,
                         int32_t *perm, int32_t *order, void *ws, size_t ws_bytes) {
    if (n <= 0 || !row_ptr || !col_idx || !perm || !order || !ws) return OASIS_EINVAL;
    hipStream_t s = as_stream(stream);
    Carver c(ws, ws_bytes);
    RcmWs r;
    carve_rcm(c, n, r);
    if (!c.ok) return OASIS_EWORKSPACE;
    OASIS_TRY(fill_i(s, n, r.pos, -1));
    int placed = 0, batch = kLevels;
    while (placed < n) {
        long long key = 0;
        OASIS_TRY(rcm_minkey(s, n, nullptr, row_ptr, r.pos, r.keyp, &key));
        int root = (int)(key & 0xffffffffll);
        int depth = 0, x = 0;
        OASIS_TRY(rcm_levels(s, n, row_ptr, col_idx, r, root, &batch, &depth, &x));
        while (true) {
            int dx = 0, xx = 0;
            OASIS_TRY(rcm_levels(s, n, row_ptr, col_idx, r, x, &batch, &dx, &xx));
            if (dx > depth) {
                root = x;
                depth = dx;
                x = xx;
            } else {
                break;
            }
        }
        // Cuthill-McKee sequence of this component, level by level
        OASIS_TRY(fill_i(s, n, r.claim, -1));
        // r.grp is the sequence; levels are contiguous ranges of it
        int *cm = r.grp, *newl = r.lst[0], *par = r.lst[1], *grp = r.dist;
        hipLaunchKernelGGL(k_level_root, dim3(1), dim3(1), 0, s, root, placed, r.claim, cm, r.pos, r.lev);
        OASIS_TRY_LAUNCH();
        auto level = [&](int j) -> int {
            const dim3 g(kLevelGrid), b(kBlock);
            hipLaunchKernelGGL(k_bfs_expand, g, b, 0, s, j, cm, row_ptr, col_idx, r.pos, r.claim,
                               static_cast<int *>(nullptr), newl, r.cnt, r.fillc, r.lev);
            OASIS_TRY_LAUNCH();
            hipLaunchKernelGGL(k_cm_parent, g, b, 0, s, j, r.lev, newl, row_ptr, col_idx, r.pos, par, r.cnt);
            OASIS_TRY_LAUNCH();
            hipLaunchKernelGGL(k_cm_offsets, dim3(1), dim3(1024), 0, s, j, r.lev, r.cnt, r.off);
            OASIS_TRY_LAUNCH();
            hipLaunchKernelGGL(k_cm_group, g, b, 0, s, j, r.lev, newl, par, r.off, r.fillc, grp);
            OASIS_TRY_LAUNCH();
            hipLaunchKernelGGL(k_cm_place, g, b, 0, s, j, r.lev, newl, par, r.off, r.cnt, grp, row_ptr, r.pos, cm);
            OASIS_TRY_LAUNCH();
            return OASIS_OK;
        };
        int first = 0, size = 0;
        OASIS_TRY(rcm_batches(s, r, level, &batch, &depth, &first, &size));
        placed = first + size;
    }
    hipLaunchKernelGGL(k_rcm_finish, dim3(grid_for(n, kBlock, 8192)), dim3(kBlock), 0, s, n, r.pos,
                       r.grp, perm, order);
    OASIS_TRY_LAUNCH();
    OASIS_TRY_HIP(hipStreamSynchronize(s));
    return OASIS_OK;
}

extern "C" int oasis_relabel(void *stream, int32_t count, const int32_t *in, const int32_t *perm,
                             int32_t *out) {
    if (count < 0 || (count > 0 && (!in || !perm || !out))) return OASIS_EINVAL;
    if (count == 0) return OASIS_OK;
    hipLaunchKernelGGL(k_relabel, dim3(grid_for(count, kBlock, 8192)), dim3(kBlock), 0,
                       as_stream(stream), count, in, perm, out);
    OASIS_TRY_LAUNCH();
    return OASIS_OK;
}
