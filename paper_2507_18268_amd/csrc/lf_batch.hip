// Batched form: one persistent kernel over a task table of independent
// problems (mesh, DT, dt, boundary conditions, T).
//
// Each workgroup takes the next task from the table (an integer counter) and
// runs all of its time steps alone: assembly in FP64 with an FP32 copy of
// the coefficients, then the precision form's refinement (FP64 true residual
// and update, FP32 inner PCG with FP64 dot products, alpha and beta).  Phases
// are separated by workgroup barriers only; no workgroup ever waits for
// another, so the grid always drains.  Every sum runs in a fixed order inside
// the workgroup, so a problem's result does not depend on which other
// problems share the launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "lf_solver.h"

namespace lf {

struct BatchTask {
    // mesh (sliced row layout and geometry)
    const int32_t *soff, *scol, *sface;
    const uint8_t *rlen;
    const double *V, *mag_sf, *delta;
    const double *emag_sf, *edelta;   // per entry of the row layout, or null
    const int32_t *bface_start, *bface_list, *bface_patch;
    const double *bmag_sf, *bdelta;
    const int32_t *patch_type;
    const double *patch_value;
    // problem
    double *T, *coef, *diagB, *srcB;
    double *bic, *bbc;     // [n_bfaces] boundary coefficients in the order of bface_list
    double *t64;           // 1 / sqrt(diagB)
    float *coef32, *s32, *t32, *r32, *p32, *q32, *d32;
    double *snap;          // [n_steps][n] copies of T after each step (mesh cell order), or null
    const int32_t *iperm;  // mesh cell of each solver row, or null (same order)
    // band layout of the problem's coefficients (nb = 3; 0: sliced row layout)
    const double *band_mag_sf, *band_delta;
    int32_t nb, band_d[kMaxBands];
    double DT, dt, tol, rel_tol, inner_tol;
    int32_t n, n_bfaces, max_iter, max_outer;
};

// tightening of the refinement target, as in the single-problem precision form
constexpr double kBatchTighten = 0.1;

template <int BS>
__device__ __forceinline__ double bsum1(double v) {
    double a[1] = {v};
    block_sum<BS, 1>(a);
    return a[0];
}

template <int BS>
__device__ __forceinline__ void bsum2(double &a0, double &a1) {
    double a[2] = {a0, a1};
    block_sum<BS, 2>(a);
    a0 = a[0];
    a1 = a[1];
}

// Forms of the kernel, chosen for a launch by its largest problem (the results are
// bitwise the same in each).
//  kSmall: few rows per thread, one row per group (two with 256 threads) and fewer
//    registers, so that more workgroups share a CU.  The large form's groups of
//    up to 16 rows reach past the end of a small problem, and the rows there cost
//    as much as real ones: 1024 requests of 8^3 to 12^3 with 256, 512, 1024 threads
//    1.08, 1.25, 1.47 ms in this form, 1.64, 2.02, 1.94 in the large one; at 4096 rows
//    both take the same (16^3, 512 threads 3.3 ms).
//  kLarge: the others of up to kNearRows rows.
//  kFar: beyond.  Up to kNearRows rows a row's byte offset in any array fits the 32
//    bits of an access's offset register, the rows that a last group reaches past
//    the end (at most 2^14) among them.  Addresses good for any row would cost
//    1-2% with 512 threads and 9-18% with 1024, so larger problems go one row after
//    the other.
// Kernels of their own, since beside the far form in one kernel the large ran 2% slower.
enum BatchForm : int { kLarge, kSmall, kFar };
constexpr int32_t kSmallRows = 4096, kNearRows = (1 << 28) - (1 << 14);

// fn(rows) for the thread's groups in order.  A group is an inner one if all its
// rows are at least `halo` rows from both ends.
template <int BS, int G, BatchForm kForm, class Fn>
__device__ __forceinline__ void each_group(int32_t n, int32_t halo, Fn &&fn) {
    static_assert(G * BS <= 1 << 14, "kNearRows leaves room for one group");
    for (int32_t i = 0; i < n; i += G * BS) {
        const uint32_t c0 = static_cast<uint32_t>(i) + threadIdx.x;
        if (kForm != kFar) __builtin_assume(c0 < (1u << 28));
        if (i >= halo && i + G * BS <= n - halo)
            fn(RowGroup<BS, G, true>{c0, n - 1});
        else
            fn(RowGroup<BS, G, false>{c0, n - 1});
    }
}

// y = acc + sum of the rows' entries
template <int BS, int G, bool kIn, class T>
__device__ __forceinline__ void group_dot(const BandLayout<3> &L, const RowGroup<BS, G, kIn> &g,
                                          const T *__restrict__ coef, const T *__restrict__ x, const T (&acc)[G],
                                          T (&y)[G]) {
    T a[G][6], xv[G][6];
    group_entries(L, g, coef, MemVec<T>{x}, a, xv);
#pragma unroll
    for (int u = 0; u < G; ++u) {
        y[u] = acc[u];
#pragma unroll
        for (int j = 0; j < 6; ++j) y[u] = mul_add(a[u][j], xv[u][j], y[u]);
    }
}

template <int BS, int G, bool kIn, class T>
__device__ __forceinline__ void group_dot(const SellLayout &L, const RowGroup<BS, G, kIn> &g,
                                          const T *__restrict__ coef, const T *__restrict__ x, const T (&acc)[G],
                                          T (&y)[G]) {
#pragma unroll
    for (int u = 0; u < G; ++u) y[u] = layout_dot(L, g.row(u), coef, x, acc[u]);
}

// Assembly of the group's rows: lap_diag, and y = sum a_j x_j, sa = sum a_j of
// the row's off-diagonal entries; the coefficients are stored.
template <int BS, int G, bool kIn>
__device__ __forceinline__ void group_assemble(const BandLayout<3> &L, const RowGroup<BS, G, kIn> &g, double DT,
                                               const double *__restrict__ x, double *__restrict__ coef,
                                               double (&lap)[G], double (&a)[G][6], double (&xv)[G][6]) {
    double dl[G][6];
    group_entries(L, g, L.mag_sf, MemVec<double>{x}, a, xv);
#pragma unroll
    for (int u = 0; u < G; ++u) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int k = 2 - j;
            if constexpr (kIn) {
                dl[u][j] = g.at(L.delta + static_cast<int64_t>(k) * L.n, u, -L.d[k]);
            } else {
                const int32_t c = g.row(u);
                dl[u][j] = L.delta[static_cast<int64_t>(k) * L.n + (c >= L.d[k] ? c - L.d[k] : L.n - 1)];
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) dl[u][3 + k] = g.at(L.delta + static_cast<int64_t>(k) * L.n, u);
    }
#pragma unroll
    for (int u = 0; u < G; ++u) {
        lap[u] = 0.0;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const double up = dl[u][j] * (DT * a[u][j]);
            a[u][j] = -up;
            lap[u] -= up;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) g.set(coef + static_cast<int64_t>(k) * L.n, u, a[u][3 + k]);
    }
}

// FP32 coefficients of the scaled matrix, a_cn t_c t_n, of the group's rows
template <int BS, int G, bool kIn>
__device__ __forceinline__ void group_scale(const BandLayout<3> &L, const RowGroup<BS, G, kIn> &g,
                                            const float *__restrict__ t32, const double *__restrict__ coef,
                                            float *__restrict__ coef32) {
    double a[G][3];
    float tc[G], tn[G][3];
#pragma unroll
    for (int u = 0; u < G; ++u) {
        tc[u] = g.at(t32, u);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            a[u][k] = g.at(coef + static_cast<int64_t>(k) * L.n, u);
            if constexpr (kIn) {
                tn[u][k] = g.at(t32, u, L.d[k]);
            } else {
                const int32_t c = g.row(u);
                tn[u][k] = t32[c < L.n - L.d[k] ? c + L.d[k] : c];     // a slot without a face holds 0
            }
        }
    }
#pragma unroll
    for (int u = 0; u < G; ++u)
#pragma unroll
        for (int k = 0; k < 3; ++k)
            g.set(coef32 + static_cast<int64_t>(k) * L.n, u,
                  static_cast<float>(a[u][k] * (static_cast<double>(tc[u]) * static_cast<double>(tn[u][k]))));
}

template <int BS, int G, bool kIn>
__device__ __forceinline__ void group_scale(const SellLayout &L, const RowGroup<BS, G, kIn> &g,
                                            const float *__restrict__ t32, const double *__restrict__ coef,
                                            float *__restrict__ coef32) {
    for (int u = 0; u < G; ++u) {
        if (!g.ok(u)) continue;
        const int32_t c = g.row(u), len = L.mr.rlen[c];
        const double tc = t32[c];
        int32_t idx = row_base(L.mr, c);
        for (int32_t j = 0; j < len; ++j, idx += kSlice)
            coef32[idx] = static_cast<float>(coef[idx] * (tc * static_cast<double>(t32[L.mr.scol[idx]])));
    }
}

// One problem's steps.  The inner FP32 solve is the precision form's: CG on the
// matrix scaled to unit diagonal (t = 1/sqrt(diagB), As = t A t with t rounded to
// FP32, rs = t r, d = t y), whose iterates are those of the diagonally
// preconditioned CG of A d = r; it stops on the L1 norm of A's residual,
// sum s|rs| with s = sqrt(diagB).  r and y are scaled with t in FP64: rounded, it
// left T up to 13% further from the exact step at the same residual (16^3 to 24^3,
// against 6% nearer than CG on the unscaled matrix now) for 2 to 4% of the time.
//
// What bounds it is what one workgroup's CU can fetch past its L1: 32 bytes per
// clock, 75 GB/s, whatever level answers (the 68 bytes per row of an inner
// iteration on memory-resident vectors took 50 us at 32^3).  So the inner
// vectors live in the LDS, as many of p (which the neighbours read too), r, q
// and y as it holds (kLds of them, from the problem's size alone), and the
// start of a pass (rs, its sums) is formed where the FP64 residual is.  A
// vector kept in memory takes the same rows in the same order with the same
// expressions, so its place does not change a bit.
//
// The task's arrays are distinct allocations: taking them into __restrict__
// locals lets the compiler overlap the loads of several rows of a loop.
template <int BS, int kLds, BatchForm kForm, class Lay>
__device__ __forceinline__ void solve_task(const BatchTask &tk, const Lay &L, int32_t n_steps,
                                           lf_solve_stats *__restrict__ stats, float *lds) {
    const int32_t n = tk.n;
    const double *__restrict__ V = as_global(tk.V);
    const int32_t *__restrict__ bface_start = as_global(tk.bface_start);
    const int32_t *__restrict__ bface_list = as_global(tk.bface_list);
    double *__restrict__ T = as_global(tk.T);
    double *__restrict__ coef = as_global(tk.coef);
    double *__restrict__ diagB = as_global(tk.diagB);
    double *__restrict__ srcB = as_global(tk.srcB);
    double *__restrict__ ic = as_global(tk.bic);
    double *__restrict__ bc = as_global(tk.bbc);
    float *__restrict__ coef32 = as_global(tk.coef32);
    float *__restrict__ s32 = as_global(tk.s32);
    float *__restrict__ t32 = as_global(tk.t32);
    double *__restrict__ t64 = as_global(tk.t64);
    float *__restrict__ p = kLds > 0 ? lds : as_global(tk.p32);
    float *__restrict__ r32 = kLds > 1 ? lds + n : as_global(tk.r32);
    float *__restrict__ q32 = kLds > 2 ? lds + 2 * n : as_global(tk.q32);
    float *__restrict__ d32 = kLds > 3 ? lds + 3 * n : as_global(tk.d32);
    const int32_t *__restrict__ bface_patch = as_global(tk.bface_patch);
    const int32_t *__restrict__ patch_type = as_global(tk.patch_type);
    const double *__restrict__ patch_value = as_global(tk.patch_value);
    const double *__restrict__ bmag_sf = as_global(tk.bmag_sf);
    const double *__restrict__ bdelta = as_global(tk.bdelta);
    const int32_t tid = static_cast<int32_t>(threadIdx.x);
    const double rdt = 1.0 / tk.dt;
    const double DT = tk.DT;
    // Rows of a group, per phase.  A load that misses the L1 comes back after
    // about a microsecond and the next group's loads are not issued before: as
    // many rows as the registers (131072 / BS per thread) hold loads for, in
    // the FP32 vector updates (kG), the FP32 product (kGP), the FP64 product
    // (kG64) and the assembly (kGA).  The other forms: see BatchForm.
    constexpr int kFew = kForm == kSmall && BS == 256 ? 2 : 1;
    constexpr int kG = kForm != kLarge ? kFew : BS == 1024 ? 8 : 16, kGP = kForm != kLarge ? kFew : BS == 1024 ? 4 : 8;
    constexpr int kG64 = kForm != kLarge ? 1 : BS == 1024 ? 2 : 4, kGA = kForm != kLarge || BS == 1024 ? 1 : 4;
    constexpr bool kBand = !std::is_same_v<Lay, SellLayout>;
    int32_t halo = n;                 // rows between a row and its farthest neighbour (rows: unknown)
    if constexpr (kBand) halo = L.d[2];
    // sum of x0 = T; the later steps' is taken with the last residual
    double sx = 0.0;
    each_group<BS, kG, kForm>(n, 0, [&](const auto &g) {
        double x[kG];
#pragma unroll
        for (int u = 0; u < kG; ++u) x[u] = g.at(T, u);
#pragma unroll
        for (int u = 0; u < kG; ++u) sx += g.ok(u) ? x[u] : 0.0;
    });
    // boundary coefficients, in the order in which a row reads its faces'
    for (int32_t i = tid; i < tk.n_bfaces; i += BS) {
        const int32_t b = bface_list[i];
        const int32_t pt = bface_patch[b];
        const bool fixed = patch_type[pt] == LF_BC_FIXED_VALUE;
        const double f = DT * bmag_sf[b], dl = bdelta[b];
        ic[i] = fixed ? f * dl : 0.0;
        bc[i] = fixed ? f * (dl * patch_value[pt]) : 0.0;
    }
    sx = bsum1<BS>(sx);
    for (int32_t step = 0; step < n_steps; ++step) {
        const double x_avg = sx / static_cast<double>(n);
        // ---- assembly (FP64), r0 = b - A x0, normalisation terms
        double a_r = 0.0, a_nf = 0.0;
        // the start of a refinement pass from a row's FP64 residual: rs, which is
        // the first direction too, y = 0, and the terms of sum s|rs| and rs.rs
        double s_r = 0.0, s_wr = 0.0;
        auto start_row = [&](int32_t c, double rc, float s, double t) {
            const float rs = static_cast<float>(rc * t);
            s_r = mul_add(static_cast<double>(s), fabs(static_cast<double>(rs)), s_r);
            s_wr = mul_add(static_cast<double>(rs), static_cast<double>(rs), s_wr);
            p[c] = rs;
            r32[c] = rs;
            d32[c] = 0.0f;
        };
        // one row from its off-diagonal entries: off(ax, sa) adds sum a_j x_j
        // and sum a_j in entry order
        auto finish_row = [&](int32_t c, double v, double xc, double lap_diag, double bd, double bs, auto &&off) {
            const double db = (rdt * v - lap_diag) + bd, sb = (rdt * xc) * v + bs;
            diagB[c] = db;
            srcB[c] = sb;
            const double s = sqrt(db);
            const double t = 1.0 / s;
            const float sf = static_cast<float>(s);
            s32[c] = sf;
            t32[c] = static_cast<float>(t);
            t64[c] = t;
            double ax = db * xc, sa = db;
            off(ax, sa);
            const double rc = sb - ax;
            start_row(c, rc, sf, t);
            const double pa = sa * x_avg;
            a_r += fabs(rc);
            a_nf += fabs(ax - pa) + fabs(sb - pa);
        };
        if constexpr (kBand) {
            each_group<BS, kGA, kForm>(n, halo, [&](const auto &g) {
                double a[kGA][6], xv[kGA][6], lap[kGA], v[kGA], xc[kGA], bd[kGA], bs[kGA];
                int32_t b0[kGA], b1[kGA];
#pragma unroll
                for (int u = 0; u < kGA; ++u) {
                    b0[u] = g.at(bface_start, u);
                    b1[u] = g.at(bface_start, u, 1);
                    v[u] = g.at(V, u);
                    xc[u] = g.at(T, u);
                }
                group_assemble(L, g, DT, T, coef, lap, a, xv);
                // the rows' boundary faces side by side: one load's wait for all
#pragma unroll
                for (int u = 0; u < kGA; ++u) bd[u] = bs[u] = 0.0;
                for (int32_t t = 0;; ++t) {
                    bool more = false;
                    double di[kGA], si[kGA];
#pragma unroll
                    for (int u = 0; u < kGA; ++u) {
                        const bool has = b0[u] + t < b1[u];
                        more = more || has;
                        di[u] = has ? ic[b0[u] + t] : 0.0;
                        si[u] = has ? bc[b0[u] + t] : 0.0;
                    }
                    if (!more) break;
#pragma unroll
                    for (int u = 0; u < kGA; ++u) {
                        bd[u] += di[u];
                        bs[u] += si[u];
                    }
                }
#pragma unroll
                for (int u = 0; u < kGA; ++u)
                    if (g.ok(u))
                        finish_row(g.row(u), v[u], xc[u], lap[u], bd[u], bs[u], [&](double &ax, double &sa) {
#pragma unroll
                            for (int j = 0; j < 6; ++j) {
                                ax += a[u][j] * xv[u][j];
                                sa += a[u][j];
                            }
                        });
            });
        } else {
            for (int32_t c = tid; c < n; c += BS) {
                RowCoefs<Lay> rcf;
                const double lap_diag = assemble_coefs<false>(L, c, DT, coef, nullptr, rcf);
                double bd = 0.0, bs = 0.0;
                for (int32_t i = bface_start[c]; i < bface_start[c + 1]; ++i) {
                    bd += ic[i];
                    bs += bc[i];
                }
                finish_row(c, V[c], T[c], lap_diag, bd, bs,
                           [&](double &ax, double &sa) { row_amul_sum(L, c, coef, rcf, T, ax, sa); });
            }
        }
        {
            double a[4] = {a_r, a_nf, s_r, s_wr};
            block_sum<BS, 4, BS == 1024>(a);
            a_r = a[0];
            a_nf = a[1];
            s_r = a[2];
            s_wr = a[3];
        }
        each_group<BS, kG64, kForm>(n, halo, [&](const auto &g) { group_scale(L, g, t32, coef, coef32); });
        const double nf = a_nf + 1e-20;
        const double res0 = a_r / nf;
        double res = res0;
        int32_t n_iter = 0, n_outer = 0;
        bool nonfinite = !isfinite(res0);
        bool conv = check_conv(res0, res0, tk.tol, tk.rel_tol);
        bool tight = check_conv(res0, res0, kBatchTighten * tk.tol, kBatchTighten * tk.rel_tol);
        // ---- refinement passes
        while (!nonfinite && !tight && n_outer < tk.max_outer && n_iter < tk.max_iter) {
            __syncthreads();          // coef32 of the first pass, p of every pass
            const double target = fmax(tk.inner_tol * s_r, 0.5 * kBatchTighten * tk.tol * nf);
            double wArA = s_wr;
            double beta = 0.0;
            bool inner_done = (s_r <= target) || !(s_wr > 0.0);
            int32_t inner_iter = 0;
            while (!inner_done) {
                if (inner_iter > 0) {          // p = rs in the first iteration
                    const float fb = static_cast<float>(beta);
                    each_group<BS, kG, kForm>(n, 0, [&](const auto &g) {
                        float rs[kG], pc[kG];
#pragma unroll
                        for (int u = 0; u < kG; ++u) {
                            rs[u] = g.at(r32, u);
                            pc[u] = g.at(p, u);
                        }
#pragma unroll
                        for (int u = 0; u < kG; ++u) g.set(p, u, mul_add(fb, pc[u], rs[u]));
                    });
                    __syncthreads();
                }
                double s_pq = 0.0;
                each_group<BS, kGP, kForm>(n, halo, [&](const auto &g) {
                    float pc[kGP], qc[kGP];
#pragma unroll
                    for (int u = 0; u < kGP; ++u) pc[u] = g.at(p, u);
                    group_dot(L, g, coef32, p, pc, qc);
#pragma unroll
                    for (int u = 0; u < kGP; ++u) {
                        const float q = g.ok(u) ? qc[u] : 0.0f;
                        g.set(q32, u, q);
                        s_pq = mul_add(static_cast<double>(q), static_cast<double>(pc[u]), s_pq);
                    }
                });
                const double pq = bsum1<BS>(s_pq);
                if (!isfinite(pq)) { nonfinite = true; break; }
                if (!(fabs(pq) > 0.0)) break;
                const double alpha = wArA / pq;
                const float fa = static_cast<float>(alpha);
                double u_r = 0.0, u_wr = 0.0;
                each_group<BS, kG, kForm>(n, 0, [&](const auto &g) {
                    float sc[kG], pc[kG], rs[kG], q[kG], y[kG];
#pragma unroll
                    for (int u = 0; u < kG; ++u) {
                        sc[u] = g.at(s32, u);
                        pc[u] = g.at(p, u);
                        q[u] = g.at(q32, u);
                        rs[u] = g.at(r32, u);
                        y[u] = g.at(d32, u);
                    }
#pragma unroll
                    for (int u = 0; u < kG; ++u) {
                        rs[u] = mul_add(-fa, q[u], rs[u]);
                        g.set(r32, u, rs[u]);
                        g.set(d32, u, mul_add(fa, pc[u], y[u]));
                    }
#pragma unroll
                    for (int u = 0; u < kG; ++u) {
                        const double rd = g.ok(u) ? static_cast<double>(rs[u]) : 0.0;
                        u_r = mul_add(static_cast<double>(sc[u]), fabs(rd), u_r);
                        u_wr = mul_add(rd, rd, u_wr);
                    }
                });
                bsum2<BS>(u_r, u_wr);
                ++inner_iter;
                ++n_iter;
                if (!isfinite(u_r) || !isfinite(u_wr)) { nonfinite = true; break; }
                if (u_r <= target || n_iter >= tk.max_iter || !(u_wr > 0.0)) {
                    inner_done = true;
                } else {
                    beta = u_wr / wArA;
                    wArA = u_wr;
                }
            }
            if (nonfinite) break;
            // T += d, then the FP64 true residual (and the sum of T)
            each_group<BS, kG, kForm>(n, 0, [&](const auto &g) {
                double x[kG], tc[kG];
                float y[kG];
#pragma unroll
                for (int u = 0; u < kG; ++u) {
                    y[u] = g.at(d32, u);
                    x[u] = g.at(T, u);
                    tc[u] = g.at(t64, u);
                }
#pragma unroll
                for (int u = 0; u < kG; ++u) g.set(T, u, x[u] + static_cast<double>(y[u]) * tc[u]);
            });
            __syncthreads();
            double o_r = 0.0, o_x = 0.0;
            s_r = s_wr = 0.0;
            each_group<BS, kG64, kForm>(n, halo, [&](const auto &g) {
                double xc[kG64], ax[kG64], b[kG64], y[kG64], tc[kG64];
                float sc[kG64];
#pragma unroll
                for (int u = 0; u < kG64; ++u) {
                    xc[u] = g.at(T, u);
                    ax[u] = g.at(diagB, u);
                    b[u] = g.at(srcB, u);
                    sc[u] = g.at(s32, u);
                    tc[u] = g.at(t64, u);
                }
#pragma unroll
                for (int u = 0; u < kG64; ++u) ax[u] *= xc[u];
                group_dot(L, g, coef, T, ax, y);
#pragma unroll
                for (int u = 0; u < kG64; ++u) {
                    if (!g.ok(u)) continue;
                    const double rc = b[u] - y[u];
                    start_row(g.row(u), rc, sc[u], tc[u]);
                    o_r += fabs(rc);
                    o_x += xc[u];
                }
            });
            {
                double a[4] = {o_r, o_x, s_r, s_wr};
                block_sum<BS, 4, BS == 1024>(a);
                o_r = a[0];
                o_x = a[1];
                s_r = a[2];
                s_wr = a[3];
            }
            sx = o_x;
            res = o_r / nf;
            ++n_outer;
            nonfinite = !isfinite(res);
            conv = check_conv(res, res0, tk.tol, tk.rel_tol);
            tight = check_conv(res, res0, kBatchTighten * tk.tol, kBatchTighten * tk.rel_tol);
        }
        if (tk.snap) {
            double *__restrict__ out = as_global(tk.snap) + static_cast<int64_t>(step) * n;
            const int32_t *__restrict__ ip = as_global(tk.iperm);
            each_group<BS, kG, kForm>(n, 0, [&](const auto &g) {
                double x[kG];
#pragma unroll
                for (int u = 0; u < kG; ++u) x[u] = g.at(T, u);
#pragma unroll
                for (int u = 0; u < kG; ++u)
                    if (g.ok(u)) out[ip ? ip[g.row(u)] : g.row(u)] = x[u];
            });
        }
        if (tid == 0) {
            lf_solve_stats st;
            st.initial_residual = res0;
            st.final_residual = res;
            st.n_iter = n_iter;
            st.converged = conv ? 1 : 0;
            st.singular = 0;
            st.nonfinite = nonfinite ? 1 : 0;
            st.n_outer = n_outer;
            st.reserved = 0;
            st.assemble_ms = 0.0;
            st.solve_ms = 0.0;
            stats[step] = st;
        }
        __syncthreads();
        if (nonfinite) {
            for (int32_t s2 = step + 1 + tid; s2 < n_steps; s2 += BS) {
                lf_solve_stats st{};
                st.nonfinite = 1;
                stats[s2] = st;
            }
            return;
        }
    }
}

// LDS vectors of a problem of n rows in the band layout: as many of the four as
// fit
__host__ __device__ inline int lds_vectors(int32_t n) {
    constexpr int32_t kRows = 39 * 1024;     // 156 KiB of the CU's 160; the rest is for the sums
    return n > kRows ? 0 : kRows / n < 4 ? kRows / n : 4;
}

template <int BS, BatchForm kForm>
__global__ void __launch_bounds__(BS) k_batch(const BatchTask *__restrict__ tasks, int32_t n_tasks,
                                             int32_t *__restrict__ counter, int32_t n_steps,
                                             lf_solve_stats *__restrict__ stats) {
    extern __shared__ float lds[];
    __shared__ int32_t s_task;
    for (;;) {
        if (threadIdx.x == 0) s_task = atomicAdd(counter, 1);
        __syncthreads();
        const int32_t t = s_task;
        __syncthreads();
        if (t >= n_tasks) return;
        const BatchTask &tk = tasks[t];
        lf_solve_stats *st = stats + static_cast<int64_t>(t) * n_steps;
        if (tk.nb == 3) {
            BandLayout<3> L;
            L.n = tk.n;
#pragma unroll
            for (int k = 0; k < 3; ++k) L.d[k] = tk.band_d[k];
            L.mag_sf = as_global(tk.band_mag_sf);
            L.delta = as_global(tk.band_delta);
            if constexpr (kForm == kFar) {
                solve_task<BS, 0, kForm>(tk, L, n_steps, st, nullptr);
            } else if constexpr (kForm == kSmall) {
                solve_task<BS, 4, kForm>(tk, L, n_steps, st, lds);
            } else {
                switch (lds_vectors(tk.n)) {
                    case 0: solve_task<BS, 0, kForm>(tk, L, n_steps, st, nullptr); break;
                    case 1: solve_task<BS, 1, kForm>(tk, L, n_steps, st, lds); break;
                    case 2: solve_task<BS, 2, kForm>(tk, L, n_steps, st, lds); break;
                    case 3: solve_task<BS, 3, kForm>(tk, L, n_steps, st, lds); break;
                    default: solve_task<BS, 4, kForm>(tk, L, n_steps, st, lds); break;
                }
            }
        } else {
            const SellLayout L{MeshRows{as_global(tk.soff), as_global(tk.scol), as_global(tk.sface),
                                        as_global(tk.rlen)},
                               as_global(tk.mag_sf), as_global(tk.delta), as_global(tk.emag_sf),
                               as_global(tk.edelta)};
            solve_task<BS, 0, kForm>(tk, L, n_steps, st, nullptr);
        }
    }
}

__global__ void k_zero_counter(int32_t *counter) { *counter = 0; }

}  // namespace lf

using namespace lf;

struct lf_batch {
    int32_t max_tasks = 0, max_steps = 0;
    hipStream_t stream = nullptr;
    BatchTask *d_tasks = nullptr;
    int32_t *d_counter = nullptr;
    lf_solve_stats *d_stats = nullptr;
    BatchTask *h_tasks = nullptr;          // pinned staging of the task table
    lf_solve_stats *h_stats = nullptr;     // pinned
    hipEvent_t done = nullptr, start = nullptr;
    int32_t last_n = 0, last_steps = 0;
    bool in_flight = false;
    int device = 0;
};

// the kernel with the LDS of the launch's largest need (above 64 KiB it has to
// be allowed first)
template <int BS>
static lf_status launch_batch(BatchForm form, int32_t lds_rows, int32_t grid, int32_t n, int32_t n_steps, lf_batch *b,
                              hipStream_t s) {
    const int lds = form != kFar ? static_cast<int>(sizeof(float)) * lds_rows : 0;
    auto kern = form == kFar ? k_batch<BS, kFar> : form == kSmall ? k_batch<BS, kSmall> : k_batch<BS, kLarge>;
    if (lds > (48 << 10))
        LF_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   156 << 10));
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(BS), static_cast<unsigned>(lds), s, b->d_tasks, n,
                       b->d_counter, n_steps, b->d_stats);
    return LF_OK;
}

static void carve_batch(Carver &cv, int32_t max_tasks, int32_t max_steps, lf_batch *b) {
    auto *tasks = cv.take<BatchTask>(static_cast<size_t>(max_tasks));
    auto *counter = cv.take<int32_t>(1);
    auto *stats = cv.take<lf_solve_stats>(static_cast<size_t>(max_tasks) * max_steps);
    if (b) {
        b->d_tasks = tasks;
        b->d_counter = counter;
        b->d_stats = stats;
    }
}

extern "C" {

size_t lf_batch_workspace_bytes(int32_t max_tasks, int32_t max_steps) {
    if (max_tasks < 1 || max_steps < 1) return 0;
    Carver cv(nullptr);
    carve_batch(cv, max_tasks, max_steps, nullptr);
    return cv.bytes();
}

lf_status lf_batch_create(int32_t max_tasks, int32_t max_steps, void *ws, size_t ws_bytes, void *stream,
                          lf_batch **out) {
    clear_error();
    if (!out || max_tasks < 1 || max_steps < 1) { set_error("bad argument"); return LF_EINVAL; }
    *out = nullptr;
    Carver dry(nullptr);
    carve_batch(dry, max_tasks, max_steps, nullptr);
    if (!ws || ws_bytes < dry.bytes() || (reinterpret_cast<uintptr_t>(ws) % kAlign) != 0) {
        set_error("batch workspace too small or misaligned: need %zu bytes, 256-aligned", dry.bytes());
        return LF_ENOMEM;
    }
    lf_batch *b = new (std::nothrow) lf_batch();
    if (!b) { set_error("host allocation failed"); return LF_ENOMEM; }
    b->max_tasks = max_tasks;
    b->max_steps = max_steps;
    b->stream = static_cast<hipStream_t>(stream);
    Carver cv(ws);
    carve_batch(cv, max_tasks, max_steps, b);
    hipError_t e = hipGetDevice(&b->device);
    if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void **>(&b->h_tasks), sizeof(BatchTask) * max_tasks, hipHostMallocDefault);
    if (e == hipSuccess)
        e = hipHostMalloc(reinterpret_cast<void **>(&b->h_stats),
                          sizeof(lf_solve_stats) * static_cast<size_t>(max_tasks) * max_steps, hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreate(&b->done);
    if (e == hipSuccess) e = hipEventCreate(&b->start);
    if (e != hipSuccess) {
        set_error("batch setup failed: %s", hipGetErrorString(e));
        lf_batch_destroy(b);
        return LF_EDEVICE;
    }
    *out = b;
    return LF_OK;
}

lf_status lf_batch_destroy(lf_batch *b) {
    if (!b) return LF_OK;
    if (b->in_flight && b->done) (void)hipEventSynchronize(b->done);
    if (b->h_tasks) (void)hipHostFree(b->h_tasks);
    if (b->h_stats) (void)hipHostFree(b->h_stats);
    if (b->done) (void)hipEventDestroy(b->done);
    if (b->start) (void)hipEventDestroy(b->start);
    delete b;
    return LF_OK;
}

lf_status lf_batch_launch(lf_batch *b, int32_t n, lf_problem *const *problems, double *const *snapshots,
                          int32_t n_steps, int32_t block_threads, int32_t n_workgroups) {
    clear_error();
    if (!b || n < 1 || !problems || n_steps < 1) { set_error("bad argument"); return LF_EINVAL; }
    if (n > b->max_tasks || n_steps > b->max_steps) {
        set_error("batch holds at most %d tasks x %d steps", b->max_tasks, b->max_steps);
        return LF_EINVAL;
    }
    if (b->in_flight) { set_error("previous launch not finished (lf_batch_wait / lf_batch_poll)"); return LF_ESTATE; }
    if (block_threads != 256 && block_threads != 512 && block_threads != 1024) {
        set_error("block_threads must be 256, 512 or 1024");
        return LF_EINVAL;
    }
    {
        std::vector<const lf_problem *> seen(problems, problems + n);
        std::sort(seen.begin(), seen.end());
        if (std::adjacent_find(seen.begin(), seen.end()) != seen.end()) {
            set_error("a problem is listed twice (each task writes its problem's T and vectors)");
            return LF_EINVAL;
        }
    }
    int32_t lds_rows = 0;     // the launch's LDS, in floats
    int32_t most = 0;         // rows of its largest problem
    for (int32_t i = 0; i < n; ++i) {
        const lf_problem *P = problems[i];
        if (!P) { set_error("problem %d is NULL", i); return LF_EINVAL; }
        if (problem_in_flight(P)) { set_error("problem %d: an lf_step_begin run is in flight", i); return LF_ESTATE; }
        if (P->opts.precision != LF_PREC_MIXED || P->opts.precond != LF_PC_DIAGONAL) {
            set_error("problem %d: the batched form needs LF_PREC_MIXED with the diagonal preconditioner", i);
            return LF_EINVAL;
        }
        if (P->mesh->device != b->device) { set_error("problem %d lives on another device", i); return LF_EINVAL; }
        if (P->nonorth) {
            set_error("problem %d: the batched kernel has no non-orthogonal correction", i);
            return LF_EINVAL;
        }
        const lf_mesh *m = P->mesh;
        BatchTask &t = b->h_tasks[i];
        t.soff = m->soff; t.scol = m->scol; t.sface = m->sface; t.rlen = m->rlen;
        t.V = m->V; t.mag_sf = m->mag_sf; t.delta = m->delta;
        t.emag_sf = m->emag_sf; t.edelta = m->edelta;
        t.bface_start = m->rbface_start; t.bface_list = m->rbface_list; t.bface_patch = m->bface_patch;
        t.iperm = m->iperm;
        t.bmag_sf = m->bmag_sf; t.bdelta = m->bdelta;
        t.patch_type = P->patch_type; t.patch_value = P->patch_value;
        t.T = P->T; t.coef = P->coef; t.diagB = P->diagB; t.srcB = P->srcB;
        t.bic = P->bic; t.bbc = P->bbc;
        t.t64 = P->r;
        t.coef32 = P->coef32; t.s32 = P->diag32; t.t32 = P->rD32; t.r32 = P->r32;
        t.p32 = P->p32; t.q32 = P->q32; t.d32 = P->d32;
        t.snap = snapshots ? snapshots[i] : nullptr;
        if (P->banded && m->n_bands != 3) {
            set_error("problem %d: the batched form takes the band layout of 3-band (structured 3-D) meshes "
                      "only; create it with LF_LAYOUT_ROWS", i);
            return LF_EINVAL;
        }
        t.nb = P->banded ? 3 : 0;
        for (int k = 0; k < kMaxBands; ++k) t.band_d[k] = k < m->n_bands ? m->band_d[k] : 0;
        t.band_mag_sf = m->band_mag_sf;
        t.band_delta = m->band_delta;
        t.DT = P->DT; t.dt = P->dt; t.tol = P->sp.tol; t.rel_tol = P->sp.rel_tol; t.inner_tol = P->sp.inner_tol;
        t.n = m->N; t.max_iter = P->sp.max_iter; t.max_outer = P->sp.max_outer;
        t.n_bfaces = m->B;
        if (t.nb == 3) lds_rows = std::max(lds_rows, lds_vectors(t.n) * t.n);
        most = std::max(most, t.n);
    }
    for (int32_t i = 0; i < n; ++i) problems[i]->sumx_valid = false;     // the launch rewrites T
    const BatchForm form = most > kNearRows ? kFar : most <= kSmallRows ? kSmall : kLarge;
    hipStream_t s = b->stream;
    int32_t g = n_workgroups > 0 ? std::min(n_workgroups, n) : n;
    LF_HIP(hipMemcpyAsync(b->d_tasks, b->h_tasks, sizeof(BatchTask) * n, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_zero_counter, dim3(1), dim3(1), 0, s, b->d_counter);
    LF_HIP(hipEventRecord(b->start, s));
    switch (block_threads) {
        case 256: LF_TRY(launch_batch<256>(form, lds_rows, g, n, n_steps, b, s)); break;
        case 512: LF_TRY(launch_batch<512>(form, lds_rows, g, n, n_steps, b, s)); break;
        default: LF_TRY(launch_batch<1024>(form, lds_rows, g, n, n_steps, b, s)); break;
    }
    LF_HIP(hipGetLastError());
    LF_HIP(hipMemcpyAsync(b->h_stats, b->d_stats, sizeof(lf_solve_stats) * static_cast<size_t>(n) * n_steps,
                          hipMemcpyDeviceToHost, s));
    LF_HIP(hipEventRecord(b->done, s));
    b->last_n = n;
    b->last_steps = n_steps;
    b->in_flight = true;
    return LF_OK;
}

lf_status lf_batch_poll(lf_batch *b, int32_t *finished) {
    clear_error();
    if (!b || !finished) { set_error("bad argument"); return LF_EINVAL; }
    if (!b->in_flight) { *finished = 1; return LF_OK; }
    hipError_t e = hipEventQuery(b->done);
    if (e == hipSuccess) { *finished = 1; b->in_flight = false; return LF_OK; }
    if (e == hipErrorNotReady) { *finished = 0; return LF_OK; }
    set_error("hipEventQuery failed: %s", hipGetErrorString(e));
    return LF_EDEVICE;
}

lf_status lf_batch_wait(lf_batch *b) {
    clear_error();
    if (!b) { set_error("bad argument"); return LF_EINVAL; }
    if (!b->in_flight) return LF_OK;
    LF_HIP(hipEventSynchronize(b->done));
    b->in_flight = false;
    return LF_OK;
}

lf_status lf_batch_stats(lf_batch *b, lf_solve_stats *stats, double *elapsed_ms) {
    clear_error();
    if (!b) { set_error("bad argument"); return LF_EINVAL; }
    if (b->in_flight) { set_error("launch still running"); return LF_ESTATE; }
    if (stats) std::memcpy(stats, b->h_stats, sizeof(lf_solve_stats) * static_cast<size_t>(b->last_n) * b->last_steps);
    if (elapsed_ms) {
        float ms = 0.f;
        LF_HIP(hipEventElapsedTime(&ms, b->start, b->done));
        *elapsed_ms = ms;
    }
    return LF_OK;
}

}  // extern "C"
