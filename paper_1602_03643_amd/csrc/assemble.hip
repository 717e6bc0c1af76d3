// Colour-by-colour P1 assembly into an existing CSR pattern, and the
// stand-alone sparse product.
//
// Alg. 2 of the paper re-assembles the convection matrix into the storage
// of A every step.  Here the cells of one colour share no dof, so one
// launch per colour scatters into rows that no other thread touches: no
// atomics, deterministic results.  Each block stages the element matrices
// of its 256 cells in LDS (one thread per cell computes geometry and the
// (D+1)^2 entries), then all threads cooperate on the scatter so that the
// lanes writing one row sit next to each other.
#include <algorithm>
#include <cstdlib>
#include <vector>

#include "assemble.hpp"
#include "p1.hpp"
#include "spmv.hpp"

namespace oasis {

template <int D>
__global__ __launch_bounds__(kBlock) void k_assemble(int ncell, const int *__restrict__ clist,
                                                     const double *__restrict__ X,
                                                     const int *__restrict__ cells,
                                                     const int *__restrict__ v2d,
                                                     const int *__restrict__ rp,
                                                     const int *__restrict__ ci,
                                                     double *__restrict__ out, int form,
                                                     double alpha, P3 U1, P3 U2, double c1,
                                                     double c2, int *missing) {
    constexpr int NV = D + 1;
    constexpr int NE = NV * NV;
    __shared__ double lm[kBlock * NE];
    __shared__ int ld[kBlock * NV];
    const int c0 = blockIdx.x * kBlock;
    const int nloc = min(kBlock, ncell - c0);
    const int t = threadIdx.x;
    if (t < nloc) {
        const int cell = clist[c0 + t];
        double x[NV][D];
        int dof[NV];
#pragma unroll
        for (int a = 0; a < NV; ++a) {
            const int v = cells[(long long)cell * NV + a];
            dof[a] = v2d[v];
#pragma unroll
            for (int k = 0; k < D; ++k) x[a][k] = X[(long long)v * D + k];
        }
        Elem<D> e;
        p1_element<D>(x, e);
        double ub[NV][D];
        if (form == OASIS_FORM_CONV) {
#pragma unroll
            for (int a = 0; a < NV; ++a)
#pragma unroll
                for (int k = 0; k < D; ++k)
                    ub[a][k] = c1 * U1.p[k][dof[a]] + (c2 != 0.0 ? c2 * U2.p[k][dof[a]] : 0.0);
        } else {
#pragma unroll
            for (int a = 0; a < NV; ++a)
#pragma unroll
                for (int k = 0; k < D; ++k) ub[a][k] = 0.0;
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            ld[t * NV + i] = dof[i];
#pragma unroll
            for (int j = 0; j < NV; ++j) lm[t * NE + i * NV + j] = alpha * p1_entry<D>(form, e, i, j, ub);
        }
    }
    __syncthreads();
    for (int q = t; q < nloc * NE; q += kBlock) {
        const int cl = q / NE, ij = q - cl * NE;
        const int i = ij / NV, j = ij - i * NV;
        const int row = ld[cl * NV + i], col = ld[cl * NV + j];
        const int s = rp[row], e = rp[row + 1];
        int pos = -1;
        for (int k = s; k < e; ++k)
            if (ci[k] == col) {
                pos = k;
                break;
            }
        if (pos >= 0)
            out[pos] += lm[q];
        else if (missing)
            atomicOr(missing, 1);
    }
}

int assemble_colored(hipStream_t s, const oasis_mesh *m, const int *rp, const int *ci, double *out,
                     int form, double alpha, P3 U1, P3 U2, double c1, double c2, int *missing) {
    for (int k = 0; k < m->n_colors; ++k) {
        const int a = m->color_ptr[k], b = m->color_ptr[k + 1];
        if (b <= a) continue;
        const int g = (b - a + kBlock - 1) / kBlock;
        if (m->dim == 3)
            hipLaunchKernelGGL(k_assemble<3>, dim3(g), dim3(kBlock), 0, s, b - a, m->color_cells + a,
                               m->coords, m->cells, m->vert2dof, rp, ci, out, form, alpha, U1, U2,
                               c1, c2, missing);
        else
            hipLaunchKernelGGL(k_assemble<2>, dim3(g), dim3(kBlock), 0, s, b - a, m->color_cells + a,
                               m->coords, m->cells, m->vert2dof, rp, ci, out, form, alpha, U1, U2,
                               c1, c2, missing);
        OASIS_TRY_LAUNCH();
    }
    return OASIS_OK;
}

// ---------------------------------------------------------------------------
// Assembly by rows for the stand-alone entry point with a workspace.
//
// The colours give every cell of a dof a slot of its own, so the dof -> cells
// table is one scatter without atomics: slot k of dof d holds its cell of
// colour k.  Each row then adds its cells' contributions in LDS, in ascending
// order of the cells (in that of the colours where they are more than 64), and
// writes each entry once.  The colour launches instead touch every row's lines
// once per colour: on the 97x97x73 channel 40 launches of 83 us (3.4 ms) moved
// some 8 GB; the table takes 0.32 ms here and the rows 0.30.

// colour of every cell that a class lists; classes: the host's class starts,
// by value
struct ClassPtr {
    int n, start[129];
};
__global__ __launch_bounds__(kBlock) void k_cell_colors(int ncell, ClassPtr cp, const int *__restrict__ clist,
                                                        unsigned char *__restrict__ color) {
    __shared__ int st[129];
    for (int i = threadIdx.x; i <= cp.n; i += kBlock) st[i] = cp.start[i];
    __syncthreads();
    for (int q = blockIdx.x * kBlock + threadIdx.x; q < ncell; q += gridDim.x * kBlock) {
        int lo = 0, hi = cp.n - 1;   // the last class that starts at or before q
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (st[mid] <= q)
                lo = mid;
            else
                hi = mid - 1;
        }
        const int c = clist[q];
        if (c >= 0 && c < ncell) color[c] = static_cast<unsigned char>(lo);
    }
}

// a cell that no class lists: it has no slots, and nothing is added for it
constexpr int kNoColor = 255;

template <int NV>
__global__ __launch_bounds__(kBlock) void k_slot_fill(int ncell, int w, const int *__restrict__ cells,
                                                      const int *__restrict__ v2d,
                                                      const unsigned char *__restrict__ color,
                                                      int *__restrict__ slots) {
    for (int c = blockIdx.x * kBlock + threadIdx.x; c < ncell; c += gridDim.x * kBlock) {
        const int k = color[c];
        if (k == kNoColor) continue;
#pragma unroll
        for (int a = 0; a < NV; ++a) {
            const int d = v2d[cells[(long long)c * NV + a]];
            slots[(long long)d * w + k] = c * NV + a;
        }
    }
}

// each dof's slots without the empty ones and ascending, in place (one wave
// per dof); deg[d]: their number.  Ascending, so that neighbouring rows
// read neighbouring cells at the same time: in colour order the rows took
// 732 us where 429 then did on the 97x97x73 channel.  Up to 64 slots are ranked
// from lane to lane; longer tables are only packed.
__global__ __launch_bounds__(kBlock) void k_slot_pack(int n, int w, int *slots, int *__restrict__ deg) {
    const int wl = threadIdx.x & (kWave - 1);
    for (long long d = (blockIdx.x * (long long)kBlock + threadIdx.x) / kWave; d < n;
         d += (long long)gridDim.x * (kBlock / kWave)) {
        int *row = slots + d * w;
        int at = 0;
        for (int k0 = 0; k0 < w; k0 += kWave) {
            const int v = k0 + wl < w ? row[k0 + wl] : -1;
            const unsigned long long m = __ballot(v >= 0);
            int rank = 0;
            if (w <= kWave) {
                for (unsigned long long b = m; b; b &= b - 1)
                    rank += __builtin_amdgcn_readlane(v, __builtin_ctzll(b)) < v ? 1 : 0;
            } else {
                rank = __popcll(m & ((1ull << wl) - 1ull));
            }
            if (v >= 0) row[at + rank] = v;
            at += __popcll(m);
        }
        if (wl == 0) deg[d] = at;
    }
}

// empty slots, and no cell with a colour (words of four: the array's end is
// padded)
__global__ __launch_bounds__(kBlock) void k_slot_clear(long long m, int4 *slots, int words, unsigned *color) {
    static_assert(kNoColor == 0xff, "all ones");
    const long long i0 = blockIdx.x * (long long)kBlock + threadIdx.x, step = (long long)gridDim.x * kBlock;
    for (long long i = i0; i < m; i += step) slots[i] = int4{-1, -1, -1, -1};
    for (long long i = i0; i < words; i += step) color[i] = ~0u;
}

// What the convection form needs of a vertex besides its dof, coordinates and
// u_bar, as D planes of two doubles.  Neighbouring rows gather
// neighbouring vertices, so a plane's 64 gathers lie in some 8 lines, those of
// a structure of 64 bytes per vertex in 32, four times over (450 us where the
// planes take 329; coordinates and u_bar of 24 and 32 bytes, 355).
template <int D>
__global__ __launch_bounds__(kBlock) void k_vertices(int nvert, const int *__restrict__ v2d,
                                                     const double *__restrict__ X, P3 U, double2 *__restrict__ vert) {
    for (int v = blockIdx.x * kBlock + threadIdx.x; v < nvert; v += gridDim.x * kBlock) {
        const int d = v2d[v];
        double r[2 * D];
#pragma unroll
        for (int c = 0; c < D; ++c) {
            r[c] = X[(long long)v * D + c];
            r[D + c] = U.p[c][d];
        }
#pragma unroll
        for (int q = 0; q < D; ++q) vert[(long long)q * nvert + v] = double2{r[2 * q], r[2 * q + 1]};
    }
}

// One thread per row; its entries and their columns in its column of LDS,
// found by halving (matched one by one in registers, 256 instructions a cell,
// convection on 670,000 rows took 434 us where this took 380), NC cells' loads
// in flight (four: 355) and the row's slots read NC at a time (302 us with the
// planes).
// Rows that are longer, or not in column order, add to their own entries in
// memory.  Bound by the gathers incidence -> vertices -> dofs -> coordinates
// and u_bar.
constexpr int kRowCap = 16;
template <int D, int FORM, int NC = D == 3 && FORM == OASIS_FORM_CONV ? 4 : 2>
__global__ __launch_bounds__(kBlock) void k_assemble_rows(int n, int w, const int *__restrict__ slots,
                                                          const int *__restrict__ deg,
                                                          const int *__restrict__ cells,
                                                          const int *__restrict__ v2d, int nvert,
                                                          const double *__restrict__ X,
                                                          const double2 *__restrict__ vert,
                                                          const int *__restrict__ rp,
                                                          const int *__restrict__ ci, const double *base,
                                                          double *out, double alpha, int gk) {
    constexpr int NV = D + 1;
    constexpr double mfac = 1.0 / ((D + 1) * (D + 2));
    constexpr bool kConv = FORM == OASIS_FORM_CONV;
    struct Cell {
        double x[NV][D], u[kConv ? NV : 1][D];
        int dof[NV], la;
    };
    // a thread's row: columns and sums (no other thread reads them)
    __shared__ int col[kRowCap][kBlock];
    __shared__ double a[kRowCap][kBlock];
    const RowRange<1> rr(n);
    for (long long row = rr.first + rr.gid; row < rr.last; row += rr.ngroups) {
        const int s = rp[row], len = rp[row + 1] - s;
        const int m = deg[row];
        const int *inc = slots + row * w;
        auto load = [&](int code, Cell &C) {
            const int cell = code / NV;
            C.la = code - cell * NV;
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const int v = cells[(long long)cell * NV + k];
                C.dof[k] = v2d[v];
                if constexpr (kConv) {
                    double r[2 * D];
#pragma unroll
                    for (int q = 0; q < D; ++q) {
                        const double2 p = vert[(long long)q * nvert + v];
                        r[2 * q] = p.x;
                        r[2 * q + 1] = p.y;
                    }
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        C.x[k][c] = r[c];
                        C.u[k][c] = r[D + c];
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < D; ++c) C.x[k][c] = X[(long long)v * D + c];
                }
            }
        };
        // alpha times the cell's entries (la, j)
        auto entries = [&](const Cell &C, double keep, double(&v)[NV]) {
            Elem<D> e;
            p1_element<D>(C.x, e);
            double wv[D];
#pragma unroll
            for (int c = 0; c < D; ++c) {
                if constexpr (kConv) {
                    double S = 0.0, ua = C.u[0][c];
#pragma unroll
                    for (int k = 0; k < NV; ++k) S += C.u[k][c];
#pragma unroll
                    for (int k = 1; k < NV; ++k) ua = C.la == k ? C.u[k][c] : ua;
                    wv[c] = S + ua;
                } else {
                    double ga = e.g[0][c];
#pragma unroll
                    for (int k = 1; k < NV; ++k) ga = C.la == k ? e.g[k][c] : ga;
                    wv[c] = ga;
                }
            }
            const double fac = keep * alpha * e.vol;
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                if constexpr (FORM == OASIS_FORM_MASS) {
                    v[j] = fac * mfac * (j == C.la ? 2.0 : 1.0);
                } else if constexpr (FORM == OASIS_FORM_GRAD_X) {
                    double g = e.g[j][0];
#pragma unroll
                    for (int c = 1; c < D; ++c) g = gk == c ? e.g[j][c] : g;
                    v[j] = fac * (1.0 / NV) * g;
                } else {
                    double g = 0.0;
#pragma unroll
                    for (int c = 0; c < D; ++c) g += e.g[j][c] * wv[c];
                    v[j] = fac * (kConv ? mfac : 1.0) * g;
                }
            }
        };
        const int tid = threadIdx.x;
        bool fits = len <= kRowCap;
        if (fits) {
            int last = -1;
#pragma unroll
            for (int q = 0; q < kRowCap; ++q) {
                const int c = q < len ? ci[s + q] : 0x7fffffff;
                col[q][tid] = c;
                a[q][tid] = base && q < len ? base[s + q] : 0.0;
                fits = fits && (q >= len || c > last);   // ascending
                last = c;
            }
        }
        if (fits) {
            for (int t = 0; t < m; t += NC) {
                // (a row has w slots, a multiple of NC)
                typedef int Codes __attribute__((ext_vector_type(NC)));
                const Codes code = *reinterpret_cast<const Codes *>(inc + t);
                Cell c[NC];
#pragma unroll
                for (int h = 0; h < NC; ++h) load(t + h < m ? code[h] : code[0], c[h]);
#pragma unroll
                for (int h = 0; h < NC; ++h) {
                    if (t + h >= m) break;
                    double v[NV];
                    entries(c[h], 1.0, v);
                    // the entry's place, by halving the sorted columns
                    int at[NV];
#pragma unroll
                    for (int j = 0; j < NV; ++j) at[j] = 0;
#pragma unroll
                    for (int half = kRowCap / 2; half > 0; half >>= 1)
#pragma unroll
                        for (int j = 0; j < NV; ++j) at[j] += col[at[j] + half][tid] <= c[h].dof[j] ? half : 0;
#pragma unroll
                    for (int j = 0; j < NV; ++j)
                        if (col[at[j]][tid] == c[h].dof[j]) a[at[j]][tid] += v[j];
                }
            }
#pragma unroll
            for (int q = 0; q < kRowCap; ++q)
                if (q < len) out[s + q] = a[q][tid];
        } else {
            for (int q = 0; q < len; ++q) out[s + q] = base ? base[s + q] : 0.0;
            for (int t = 0; t < m; ++t) {
                Cell c;
                double v[NV];
                load(inc[t], c);
                entries(c, 1.0, v);
#pragma unroll
                for (int j = 0; j < NV; ++j)
                    for (int q = 0; q < len; ++q)
                        if (ci[s + q] == c.dof[j]) {
                            out[s + q] += v[j];
                            break;
                        }
            }
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_axpby_copy(long long n, T *__restrict__ y,
                                                       const T *__restrict__ x, T a) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        y[i] = x ? a * x[i] : T(0);
}

int scale_copy(hipStream_t s, long long n, double *y, const double *x, double a) {
    const int g = (int)std::min<long long>((n + kBlock - 1) / kBlock, 16384);
    hipLaunchKernelGGL((k_axpby_copy<double>), dim3(g), dim3(kBlock), 0, s, n, y, x, a);
    OASIS_TRY_LAUNCH();
    return OASIS_OK;
}

template <typename T, class C>
__global__ __launch_bounds__(kBlock) void k_spmv(int n, const int *__restrict__ rp,
                                                 const int *__restrict__ ci,
                                                 const T *__restrict__ val,
                                                 const T *__restrict__ x, T *__restrict__ y, T alpha,
                                                 T beta) {
    csr_rows<T, 1, C>(
        n, rp, ci, val,
        [&](int, int c, T v, bool ok, T(&a)[1]) {
            const T t = v * x[c];
            a[0] += ok ? t : T(0);
        },
        [&](int row, int lane, T(&a)[1]) {
            if (lane == 0) y[row] = beta == T(0) ? alpha * a[0] : alpha * a[0] + beta * y[row];
        });
}

template <typename T>
static int spmv_launch(hipStream_t s, const oasis_csr *A, const T *x, T *y, T alpha, T beta) {
    const T *val = static_cast<const T *>(A->val);
    return with_cfg([&](auto c) -> int {
        using C = decltype(c);
        // one lane group per row group: the grid is not capped (no partials)
        const int g = grid_for(A->n, rows_per_block<C>(), 1 << 20);
        hipLaunchKernelGGL((k_spmv<T, C>), dim3(g), dim3(kBlock), 0, s, A->n, A->row_ptr, A->col_idx, val, x,
                           y, alpha, beta);
        OASIS_TRY_LAUNCH();
        return OASIS_OK;
    });
}

int check_csr(const oasis_csr *A) {
    if (!A || A->n <= 0 || A->nnz < 0 || !A->row_ptr || (A->nnz > 0 && (!A->col_idx || !A->val)))
        return OASIS_EINVAL;
    if (A->dtype != OASIS_F64 && A->dtype != OASIS_F32) return OASIS_EINVAL;
    if (!aligned(A->val, A->dtype == OASIS_F64 ? 8 : 4)) return OASIS_EINVAL;
    return OASIS_OK;
}

int check_mesh_colored(const oasis_mesh *m) {
    if (!m || (m->dim != 2 && m->dim != 3) || m->n_vert <= 0 || m->n_cell <= 0 || m->n_dof <= 0)
        return OASIS_EINVAL;
    if (!m->coords || !m->cells || !m->vert2dof || m->n_colors <= 0 || !m->color_ptr ||
        !m->color_cells)
        return OASIS_EINVAL;
    if (m->color_ptr[0] != 0 || m->color_ptr[m->n_colors] != m->n_cell) return OASIS_EINVAL;
    return OASIS_OK;
}

}  // namespace oasis

using namespace oasis;

extern "C" int oasis_spmv(void *stream, const oasis_csr *A, const void *x, void *y, double alpha,
                          double beta) {
    OASIS_TRY(check_csr(A));
    if (!x || !y) return OASIS_EINVAL;
    hipStream_t s = as_stream(stream);
    if (A->dtype == OASIS_F64)
        return spmv_launch<double>(s, A, static_cast<const double *>(x), static_cast<double *>(y),
                                   alpha, beta);
    return spmv_launch<float>(s, A, static_cast<const float *>(x), static_cast<float *>(y),
                              static_cast<float>(alpha), static_cast<float>(beta));
}

// The checks of the assembly entry points; u receives u_bar for FORM_CONV.
static int check_assembly(const oasis_mesh *mesh, int32_t form, const double *const *uab, const oasis_csr *base,
                          const oasis_csr *out, P3 *u) {
    OASIS_TRY(check_mesh_colored(mesh));
    OASIS_TRY(check_csr(out));
    if (out->dtype != OASIS_F64 || out->n != mesh->n_dof) return OASIS_EINVAL;
    if (form < OASIS_FORM_MASS || form > OASIS_FORM_CONV) return OASIS_EINVAL;
    if (form == OASIS_FORM_GRAD_Z && mesh->dim != 3) return OASIS_EINVAL;
    *u = P3{};
    if (form == OASIS_FORM_CONV) {
        if (!uab) return OASIS_EINVAL;
        for (int k = 0; k < mesh->dim; ++k) {
            if (!uab[k]) return OASIS_EINVAL;
            u->p[k] = uab[k];
        }
    }
    if (base) {
        OASIS_TRY(check_csr(base));
        if (base->dtype != OASIS_F64 || base->nnz != out->nnz || base->n != out->n) return OASIS_EINVAL;
    }
    return OASIS_OK;
}

extern "C" int oasis_assemble_p1(void *stream, const oasis_mesh *mesh, int32_t form,
                                 const double *const *uab, double alpha, const oasis_csr *base,
                                 oasis_csr *out) {
    P3 U1{}, U2{};
    OASIS_TRY(check_assembly(mesh, form, uab, base, out, &U1));
    hipStream_t s = as_stream(stream);
    OASIS_TRY(scale_copy(s, out->nnz, static_cast<double *>(out->val),
                         base ? static_cast<const double *>(base->val) : nullptr, 1.0));
    // entries absent from the pattern are skipped (no flag without a workspace)
    OASIS_TRY(assemble_colored(s, mesh, out->row_ptr, out->col_idx, static_cast<double *>(out->val),
                               form, alpha, U1, U2, 1.0, 0.0, nullptr));
    return OASIS_OK;
}

namespace {

struct AssembleWs {
    int w = 0;                       // slots per dof
    unsigned char *color = nullptr;
    int *slots = nullptr, *deg = nullptr;
    double2 *vert = nullptr;         // planes of vertices
};

void carve_assemble(Carver &c, const oasis_mesh *m, AssembleWs &a) {
    a.w = (m->n_colors + 3) / 4 * 4;
    a.color = c.take<unsigned char>(m->n_cell);
    a.slots = c.take<int>((size_t)m->n_dof * a.w);
    a.deg = c.take<int>(m->n_dof);
    a.vert = c.take<double2>((size_t)m->n_vert * m->dim);
}

template <int D>
int assemble_rows(hipStream_t s, const oasis_mesh *m, int form, P3 U, double alpha, const double *base, oasis_csr *out,
                  const AssembleWs &a) {
    constexpr int NV = D + 1;
    const int n = m->n_dof, nc = m->n_cell;
    ClassPtr cp{};
    cp.n = m->n_colors;
    for (int k = 0; k <= m->n_colors; ++k) cp.start[k] = m->color_ptr[k];
    const int gc = grid_for(nc, kBlock, 8192);
    const long long quads = (long long)n * a.w / 4;
    hipLaunchKernelGGL(k_slot_clear, dim3(grid_for(quads, kBlock, 8192)), dim3(kBlock), 0, s, quads,
                       reinterpret_cast<int4 *>(a.slots), (nc + 3) / 4, reinterpret_cast<unsigned *>(a.color));
    hipLaunchKernelGGL(k_cell_colors, dim3(gc), dim3(kBlock), 0, s, nc, cp, m->color_cells, a.color);
    hipLaunchKernelGGL(k_slot_fill<NV>, dim3(gc), dim3(kBlock), 0, s, nc, a.w, m->cells, m->vert2dof, a.color,
                       a.slots);
    hipLaunchKernelGGL(k_slot_pack, dim3(grid_for((long long)n * kWave, kBlock, 16384)), dim3(kBlock), 0, s, n, a.w,
                       a.slots, a.deg);
    if (form == OASIS_FORM_CONV)
        hipLaunchKernelGGL(k_vertices<D>, dim3(grid_for(m->n_vert, kBlock, 8192)), dim3(kBlock), 0, s, m->n_vert,
                           m->vert2dof, m->coords, U, a.vert);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid_for(n, kBlock, 1 << 20)), dim3(kBlock), 0, s, n, a.w, a.slots, a.deg,
                           m->cells, m->vert2dof, m->n_vert, m->coords, a.vert, out->row_ptr, out->col_idx, base,
                           static_cast<double *>(out->val), alpha, form - OASIS_FORM_GRAD_X);
    };
    if (form == OASIS_FORM_MASS)
        go(k_assemble_rows<D, OASIS_FORM_MASS>);
    else if (form == OASIS_FORM_STIFF)
        go(k_assemble_rows<D, OASIS_FORM_STIFF>);
    else if (form == OASIS_FORM_CONV)
        go(k_assemble_rows<D, OASIS_FORM_CONV>);
    else
        go(k_assemble_rows<D, OASIS_FORM_GRAD_X>);
    OASIS_TRY_LAUNCH();
    return OASIS_OK;
}

}  // namespace

extern "C" int oasis_assemble_p1_workspace_size(const oasis_mesh *mesh, size_t *bytes) {
    if (!bytes) return OASIS_EINVAL;
    OASIS_TRY(check_mesh_colored(mesh));
    if (mesh->n_colors > 128) return OASIS_EUNSUPPORTED;
    Carver c(nullptr, 0);
    AssembleWs a;
    carve_assemble(c, mesh, a);
    *bytes = c.bytes();
    return OASIS_OK;
}

extern "C" int oasis_assemble_p1_ws(void *stream, const oasis_mesh *mesh, int32_t form, const double *const *uab,
                                    double alpha, const oasis_csr *base, oasis_csr *out, void *ws, size_t ws_bytes) {
    P3 U{};
    OASIS_TRY(check_assembly(mesh, form, uab, base, out, &U));
    if (!ws || !aligned(ws, 256)) return OASIS_EINVAL;
    if (mesh->n_colors > 128) return OASIS_EUNSUPPORTED;
    Carver c(ws, ws_bytes);
    AssembleWs a;
    carve_assemble(c, mesh, a);
    if (!c.ok) return OASIS_EWORKSPACE;
    hipStream_t s = as_stream(stream);
    const double *b = base ? static_cast<const double *>(base->val) : nullptr;
    return mesh->dim == 3 ? assemble_rows<3>(s, mesh, form, U, alpha, b, out, a)
                          : assemble_rows<2>(s, mesh, form, U, alpha, b, out, a);
}
