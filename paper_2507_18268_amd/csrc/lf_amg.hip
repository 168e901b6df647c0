// Aggregation multigrid preconditioner (FP64) for meshes with the box form.
//
// The paper's conclusion names an algebraic multigrid library as the better
// alternative to the diagonal PCG.  Here the cycle is built on the box: level
// l + 1 aggregates the 2 x 2 x 2 blocks of level l (a side of odd length ends
// with a block one cell thick), every level is again a box numbered
// i + nx (j + ny k), so each level's matrix lives in the band layout and is
// applied by the same row gathers as the fine one.  Coarse matrices are the
// Galerkin products P^T A P of the piecewise-constant prolongation P, formed
// once per time step from the assembled matrix; the smoother is weighted
// Jacobi.  One application w = M r:
//   level l, right side b: x = 0; nu sweeps x += omega (b - A x) / diag;
//   b_{l+1} = the residual b - A x summed over each block; the cycle on
//   level l + 1; x += its result on every cell of the block; nu sweeps.
//   The coarsest level (at most 512 cells, or a side shorter than 3): nu_c
//   sweeps from x = 0.
// Every sum is taken in the order of the sequential definition (a block's
// cells in ascending index, a row's entries in face order), so each level's
// matrix and each application equal the sequential cycle's bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "lf_solver.h"

namespace lf {

constexpr int kAmgNu = 2;             // sweeps before and after the coarse correction
constexpr int kAmgNuC = 4;            // sweeps on the coarsest level
constexpr double kAmgOmega = 0.8;     // Jacobi weight
constexpr int64_t kAmgCoarsest = 512; // a level this small is not coarsened further
constexpr int32_t kAmgMinSide = 3;    // nor one with a side shorter than this
// a level takes the block walk from this many workgroups on (about 2 M cells;
// on smaller levels, whose launches are latency-bound, the one-row kernels
// finish sooner)
constexpr int32_t kAmgWalkMinBlocks = 1024;
static_assert(kAmgNu == 2 && kAmgNuC == 4, "the launches pair the first two sweeps; the LDS cycle alternates two iterates");

struct AmgBox {
    int32_t nx, ny, nz;
    int32_t n() const { return nx * ny * nz; }
};

static std::vector<AmgBox> amg_boxes(const lf_mesh *m) {
    std::vector<AmgBox> v{{m->box_nx, m->box_ny, m->box_nz}};
    for (;;) {
        const AmgBox b = v.back();
        if (static_cast<int64_t>(b.n()) <= kAmgCoarsest || std::min({b.nx, b.ny, b.nz}) < kAmgMinSide) break;
        v.push_back({(b.nx + 1) / 2, (b.ny + 1) / 2, (b.nz + 1) / 2});
    }
    return v;
}

static void plan_amg_walks(lf_problem *P);
static void plan_amg_tail(lf_problem *P);

void carve_amg(Carver &cv, const lf_mesh *m, lf_problem *P) {
    const std::vector<AmgBox> boxes = amg_boxes(m);
    double *t1 = cv.take<double>(static_cast<size_t>(m->N));
    double *t2 = cv.take<double>(static_cast<size_t>(m->N));
    std::vector<AmgLevel> lv;
    for (size_t l = 1; l < boxes.size(); ++l) {
        AmgLevel a;
        a.nx = boxes[l].nx;
        a.ny = boxes[l].ny;
        a.nz = boxes[l].nz;
        a.n = boxes[l].n();
        const size_t n = static_cast<size_t>(a.n);
        a.coef = cv.take<double>(3 * n);
        a.diag = cv.take<double>(n);
        a.b = cv.take<double>(n);
        a.xa = cv.take<double>(n);
        a.xb = cv.take<double>(n);
        lv.push_back(a);
    }
    if (P) {
        P->amg = lv;
        P->amg_t1 = t1;
        P->amg_t2 = t2;
        plan_amg_walks(P);
        plan_amg_tail(P);
    }
}

static BandLayout<3> box_layout(int32_t nx, int32_t ny, int32_t nz) {
    BandLayout<3> L;
    L.n = nx * ny * nz;
    L.d[0] = 1;
    L.d[1] = nx;
    L.d[2] = nx * ny;
    L.mag_sf = nullptr;
    L.delta = nullptr;
    return L;
}

// The residual b - A x summed over the cells (ascending) of coarse cell t / 8,
// by eight neighbouring lanes: lane t % 8 forms one cell's residual, and every
// lane adds the eight in order (a cell past the end of an odd side adds 0 to a
// sum that is never -0).  One thread per coarse cell ran its eight rows one
// after the other in an eighth of the wavefronts: 35.6 us for the three
// launches at 100^3, 50^3 and 25^3 cells, against 23.5.  All lanes of a wave
// call it together; past the last coarse cell (t >= 8 cn) the result is unused.
__device__ __forceinline__ double amg_block_residual(const BandLayout<3> &F, int32_t fnx, int32_t fny, int32_t fnz,
                                                     int32_t cnx, int32_t cny, int32_t cn, int32_t t,
                                                     const double *__restrict__ diag,
                                                     const double *__restrict__ coef, const double *__restrict__ b,
                                                     const double *__restrict__ x) {
    const int32_t I = t >> 3;
    const int32_t ix = I % cnx, iy = (I / cnx) % cny, iz = I / (cnx * cny);
    const int32_t fx = 2 * ix + (t & 1), fy = 2 * iy + ((t >> 1) & 1), fz = 2 * iz + ((t >> 2) & 1);
    double r = 0.0;
    if (I < cn && fx < fnx && fy < fny && fz < fnz) {
        const int32_t c = fx + fnx * (fy + fny * fz);
        const double dc = diag[c], bc = b[c];
        const double ax = layout_dot(F, c, coef, x, dc * x[c]);
        r = bc - ax;
    }
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) acc += __shfl(r, k, 8);
    return acc;
}

// coarse right side
__global__ void __launch_bounds__(kCellBlock)
k_amg_restrict(BandLayout<3> F, int32_t fnx, int32_t fny, int32_t fnz, const double *__restrict__ diag,
               const double *__restrict__ coef, const double *__restrict__ b, const double *__restrict__ x,
               int32_t cnx, int32_t cny, int32_t cn, double *__restrict__ bc, const PcgState *__restrict__ st) {
    if (st->done) return;
    const int32_t t = static_cast<int32_t>(blockIdx.x) * kCellBlock + static_cast<int32_t>(threadIdx.x);
    const double acc = amg_block_residual(F, fnx, fny, fnz, cnx, cny, cn, t, diag, coef, b, x);
    if ((t & 7) == 0 && (t >> 3) < cn) bc[t >> 3] = acc;
}

// ---------------------------------------------------------------------------
// Where a sweep takes x from: the level's iterate (MemX), the first sweep's
// values or the iterate with the coarse correction added, formed on the fly, so
// that a level's six launches (sweep, sweep, residual, correction, sweep,
// sweep) are four: below about 100 k rows each costs 4.6 us whatever it does
// (a step of the solve at 48^3 cells 2.73 ms with six, 2.20 with four).
// ---------------------------------------------------------------------------

// the first sweep's values (x = 0 + omega (b - 0) / diag)
struct AmgFirstX {
    const double *__restrict__ b;
    const double *__restrict__ diag;
    __device__ __forceinline__ Lanes<double, 2> vec(int64_t i) const {
        const Lanes<double, 2> bb = lanes_load<double, 2>(b, i), dd = lanes_load<double, 2>(diag, i);
        Lanes<double, 2> r;
#pragma unroll
        for (int w = 0; w < 2; ++w) r.v[w] = 0.0 + kAmgOmega * ((bb.v[w] - 0.0) / dd.v[w]);
        return r;
    }
    __device__ __forceinline__ double one(int64_t i) const { return 0.0 + kAmgOmega * ((b[i] - 0.0) / diag[i]); }
};

// Quotient by a fixed divisor d >= 1 for 0 <= i < 2^31 by a multiply and a
// shift (Granlund and Montgomery 1994): with s = ceil(log2 d) and
// m = floor(2^(32+s) / d) + 1, floor(i m / 2^(32+s)) = floor(i / d), since
// m d - 2^(32+s) lies in (0, d] and i < 2^32.
struct FastDiv {
    uint64_t m;
    int32_t sh;
};

inline FastDiv fast_div(uint32_t d) {
    int32_t s = 0;
    while ((uint64_t(1) << s) < d) ++s;
    return FastDiv{((uint64_t(1) << (32 + s)) / d) + 1, 32 + s};
}

__device__ __forceinline__ int64_t fdiv(int64_t i, const FastDiv &f) {
    return static_cast<int64_t>((static_cast<uint64_t>(i) * f.m) >> f.sh);
}

// the prolonged iterate x + (the coarse result of the cell's block); vec: a
// lane's two cells lie in one block (the walk's x-lines have even length)
struct AmgProlongX {
    const double *__restrict__ x;
    const double *__restrict__ xc;
    int64_t nx, ny, cnx, cny;
    FastDiv dx, dy;
    __device__ __forceinline__ int64_t block(int64_t i) const {
        const int64_t t = fdiv(i, dx), fx = i - t * nx, fz = fdiv(t, dy), fy = t - fz * ny;
        return (fx >> 1) + cnx * ((fy >> 1) + cny * (fz >> 1));
    }
    __device__ __forceinline__ Lanes<double, 2> vec(int64_t i) const {
        Lanes<double, 2> r = lanes_load<double, 2>(x, i);
        const double a = xc[block(i)];
#pragma unroll
        for (int w = 0; w < 2; ++w) r.v[w] += a;
        return r;
    }
    __device__ __forceinline__ double one(int64_t i) const { return x[i] + xc[block(i)]; }
};

// A x of row c, the diagonal term first (layout_dot's order), x from the source
template <class XS>
__device__ __forceinline__ double amg_row(const BandLayout<3> &L, int32_t c, const double *__restrict__ coef,
                                          const XS &x, double acc) {
    double a[6], xv[6];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int k = 2 - j;
        const bool ok = c >= L.d[k];
        const int32_t col = ok ? c - L.d[k] : c;
        const double v = coef[static_cast<int64_t>(k) * L.n + col];
        a[j] = ok ? v : 0.0;
        xv[j] = x.one(col);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int32_t col = c < L.n - L.d[k] ? c + L.d[k] : c;
        a[3 + k] = coef[static_cast<int64_t>(k) * L.n + c];
        xv[3 + k] = x.one(col);
    }
#pragma unroll
    for (int j = 0; j < 6; ++j) acc += a[j] * xv[j];
    return acc;
}

// y = x + omega ((b - A x) / diag), A x with the diagonal term first, one row
// per thread; kDot (level 0's last sweep, y = w, b = r): also the partial sums
// of w.r.  Bound by the launch (4.6 us) up to about 100 k rows.
template <class XS, bool kDot>
__global__ void __launch_bounds__(kCellBlock)
k_amg_sweep(SolverParams sp, BandLayout<3> L, const double *__restrict__ diag, const double *__restrict__ coef,
            const double *__restrict__ b, XS x, double *__restrict__ y, double *__restrict__ part,
            const PcgState *__restrict__ st) {
    if (st->done) return;
    const int32_t c = static_cast<int32_t>(blockIdx.x) * kCellBlock + static_cast<int32_t>(threadIdx.x);
    double acc[1] = {0.0};
    if (c < L.n) {
        const double dc = diag[c], xc = x.one(c), bc = b[c];
        const double ax = amg_row(L, c, coef, x, dc * xc);
        const double v = xc + kAmgOmega * ((bc - ax) / dc);
        y[c] = v;
        acc[0] = v * bc;
    }
    if (kDot) {
        const int slots[1] = {kPartWr};
        write_partials<1>(part, sp.grid, slots, acc);
    }
}

// ---------------------------------------------------------------------------
// The last levels of the cycle in one workgroup: what is left of the cycle from
// the first level on whose matrices and vectors, with those of all levels below
// it, fit into the LDS (56 bytes a row: 2852 rows, 13 x 13 x 13 and 7 x 7 x 7
// under a 200 x 200 x 200 box).  Bound by the chain of its passes: 19.7 us for
// those two levels, whose seven launches take 4.7 us each; a step of the solve
// at 48^3 cells 2.20 ms without, 1.94 ms with it, at 130^3 9.85 and 9.52.
// Every value is formed as by the launches it replaces, so each result is
// bitwise the same.
// ---------------------------------------------------------------------------
constexpr int kTailBlock = 1024;
constexpr int kTailLevels = 4;
constexpr int64_t kTailRows = (156 << 10) / (7 * static_cast<int64_t>(sizeof(double)));

struct AmgTail {
    int32_t count;
    int32_t nx[kTailLevels], ny[kTailLevels], nz[kTailLevels];
    int32_t off[kTailLevels];   // rows of the levels above, of the tail
    const double *coef[kTailLevels], *diag[kTailLevels];
    const double *b;
    double *x;
};

__global__ void __launch_bounds__(kTailBlock)
k_amg_tail(AmgTail T, const PcgState *__restrict__ st) {
    if (st->done) return;
    extern __shared__ double tail_mem[];
    const int32_t tid = static_cast<int32_t>(threadIdx.x);
    // the arrays of level l: the three bands, diag, b, and the two iterates
    auto at = [&](int32_t l, int32_t n, int which) { return tail_mem + 7 * T.off[l] + static_cast<int32_t>(which) * n; };
    auto rows = [&](int32_t l) { return T.nx[l] * T.ny[l] * T.nz[l]; };
    auto layout = [&](int32_t l) {
        BandLayout<3> L;
        L.n = rows(l);
        L.d[0] = 1;
        L.d[1] = T.nx[l];
        L.d[2] = T.nx[l] * T.ny[l];
        L.mag_sf = nullptr;
        L.delta = nullptr;
        return L;
    };
    for (int32_t l = 0; l < T.count; ++l) {
        const int32_t n = rows(l);
        double *m = at(l, n, 0);
        for (int32_t i = tid; i < 3 * n; i += kTailBlock) m[i] = T.coef[l][i];
        for (int32_t i = tid; i < n; i += kTailBlock) m[3 * n + i] = T.diag[l][i];
    }
    {
        const int32_t n = rows(0);
        double *b = at(0, n, 4);
        for (int32_t i = tid; i < n; i += kTailBlock) b[i] = T.b[i];
    }
    __syncthreads();
    auto first = [&](int32_t l) {   // into the first iterate
        const int32_t n = rows(l);
        const double *dg = at(l, n, 3), *b = at(l, n, 4);
        double *y = at(l, n, 5);
        for (int32_t c = tid; c < n; c += kTailBlock) y[c] = 0.0 + kAmgOmega * ((b[c] - 0.0) / dg[c]);
        __syncthreads();
    };
    auto sweep = [&](int32_t l, int from, int to) {
        const BandLayout<3> L = layout(l);
        const int32_t n = L.n;
        const double *coef = at(l, n, 0), *dg = at(l, n, 3), *b = at(l, n, 4), *x = at(l, n, from);
        double *y = at(l, n, to);
        for (int32_t c = tid; c < n; c += kTailBlock) {
            const double dc = dg[c], xc = x[c], bc = b[c];
            const double ax = amg_row(L, c, coef, MemX<double, 2>{x}, dc * xc);
            y[c] = xc + kAmgOmega * ((bc - ax) / dc);
        }
        __syncthreads();
    };
    const int32_t last = T.count - 1;
    for (int32_t l = 0; l < last; ++l) {
        first(l);
        sweep(l, 5, 6);
        const BandLayout<3> F = layout(l);
        const int32_t n = F.n, fnx = T.nx[l], fny = T.ny[l], fnz = T.nz[l], cn = rows(l + 1);
        const double *coef = at(l, n, 0), *dg = at(l, n, 3), *b = at(l, n, 4), *x = at(l, n, 6);
        double *cb = at(l + 1, cn, 4);
        for (int32_t t0 = 0; t0 < 8 * cn; t0 += kTailBlock) {
            const int32_t t = t0 + tid;
            const double acc = amg_block_residual(F, fnx, fny, fnz, T.nx[l + 1], T.ny[l + 1], cn, t, dg, coef, b, x);
            if ((t & 7) == 0 && (t >> 3) < cn) cb[t >> 3] = acc;
        }
        __syncthreads();
    }
    first(last);
    for (int k = 1; k < kAmgNuC; ++k) sweep(last, k % 2 ? 5 : 6, k % 2 ? 6 : 5);
    for (int32_t l = last - 1; l >= 0; --l) {
        const int32_t n = rows(l), fnx = T.nx[l], fny = T.ny[l], cnx = T.nx[l + 1], cny = T.ny[l + 1];
        const double *xc = at(l + 1, rows(l + 1), 6);
        double *x = at(l, n, 6);
        for (int32_t c = tid; c < n; c += kTailBlock) {
            const int32_t fx = c % fnx, fy = (c / fnx) % fny, fz = c / (fnx * fny);
            x[c] += xc[fx / 2 + cnx * (fy / 2 + cny * (fz / 2))];
        }
        __syncthreads();
        sweep(l, 6, 5);
        sweep(l, 5, 6);
    }
    const int32_t n = rows(0);
    const double *x = at(0, n, 6);
    for (int32_t c = tid; c < n; c += kTailBlock) T.x[c] = x[c];
}

// ---------------------------------------------------------------------------
// The same steps by the block walk of a box level (x-lines of even length: two
// rows per lane, 2 lines x 2 planes per thread, as the solver's product): each
// row's A x is the one-row kernels' sum term for term, so every result is
// bitwise the same.
// ---------------------------------------------------------------------------

// y = x + omega ((b - A x) / diag) with x from the source: the level's
// iterate, (AmgFirstX) the first sweep's values, so that the launch does the
// level's first two sweeps, or (AmgProlongX) the iterate with the coarse
// correction added, so that it also does the prolongation.  kDot (level 0's
// last sweep, y = w, b = r): the partial sums of w.r, one per workgroup, and
// zeros in the further entries of the slot up to the cell grid's count, which
// the reduction reads
template <class XS, bool kDot>
__global__ void __launch_bounds__(kBwBlock)
k_amg_sweep_box(SolverParams sp, BandLayout<3> L, BoxWalk bw, const double *__restrict__ diag,
                const double *__restrict__ coef, const double *__restrict__ b, XS x, double *__restrict__ y,
                double *__restrict__ part, const PcgState *__restrict__ st) {
    if (st->done) return;
    typedef Lanes<double, 2> R;
    double acc[1] = {0.0};
    const int32_t blk = walk_share(kDot);
    box_walk_xs<double, 2, false, false>(blk, L, bw, diag, coef, x, [&](int64_t c, const R &ax, const R &xc, const R &dg) {
        const R bc = lanes_load<double, 2>(b, c);
        R v;
#pragma unroll
        for (int w = 0; w < 2; ++w) v.v[w] = xc.v[w] + kAmgOmega * ((bc.v[w] - ax.v[w]) / dg.v[w]);
        *reinterpret_cast<typename R::vec *>(y + c) = typename R::vec{v.v[0], v.v[1]};
        if (kDot) {
            acc[0] += v.v[0] * bc.v[0];
            acc[0] += v.v[1] * bc.v[1];
        }
    });
    if (kDot) {
        const int slots[1] = {kPartWr};
        write_partials_at<1, kBwBlock>(part, sp.grid, blk, slots, acc);
        if (threadIdx.x == 0)
            for (int64_t j = bw.blocks + static_cast<int64_t>(blockIdx.x); j < sp.grid; j += bw.blocks)
                part[static_cast<int64_t>(kPartWr) * sp.grid + j] = 0.0;
    }
}

// k_amg_restrict on a level whose sides are all even: the walk's tiles are the
// 2 x 2 x 2 blocks (tile thread i is coarse cell i); the block's residuals are
// summed in the one-row kernel's order (z, then y, then x)
__global__ void __launch_bounds__(kBwBlock)
k_amg_restrict_box(BandLayout<3> L, BoxWalk bw, const double *__restrict__ diag, const double *__restrict__ coef,
                   const double *__restrict__ b, const double *__restrict__ x, double *__restrict__ bc,
                   const PcgState *__restrict__ st) {
    if (st->done) return;
    typedef Lanes<double, 2> R;
    const int32_t blk = walk_share(true);
    const int64_t i = static_cast<int64_t>(blk) * kBwBlock + threadIdx.x;
    // the walk visits a tile's rows line by line, within a line plane by plane:
    // the second plane of the first line waits for the first of the second
    double acc = 0.0, h0 = 0.0, h1 = 0.0;
    int call = 0;
    box_walk<double, 2, false, false>(blk, L, bw, diag, coef, x, [&](int64_t c, const R &ax, const R &, const R &) {
        const R bb = lanes_load<double, 2>(b, c);
        const double r0 = bb.v[0] - ax.v[0], r1 = bb.v[1] - ax.v[1];
        if (call == 1) {
            h0 = r0;
            h1 = r1;
        } else {
            acc += r0;
            acc += r1;
        }
        if (call == 2) {
            acc += h0;
            acc += h1;
        }
        ++call;
    });
    if (i >= static_cast<int64_t>(bw.ntiles) * bw.hx) return;
    bc[i] = acc;
}

// Galerkin coarse matrix of one block: diag = its cells' diagonals (ascending)
// then twice each face inside it (ascending face order: by cell, then +x,
// +y, +z); the coarse face to the next block in direction k = the sum of the
// fine faces crossing to it, owned by the block's cells on that side
// (ascending).  A block at the end of a direction stores 0 there.
__global__ void __launch_bounds__(kCellBlock)
k_amg_galerkin(int32_t fnx, int32_t fny, int32_t fnz, const double *__restrict__ diag,
               const double *__restrict__ coef, int32_t cnx, int32_t cny, int32_t cnz,
               double *__restrict__ cdiag, double *__restrict__ ccoef) {
    const int32_t cn = cnx * cny * cnz;
    const int32_t I = static_cast<int32_t>(blockIdx.x) * kCellBlock + static_cast<int32_t>(threadIdx.x);
    if (I >= cn) return;
    const int64_t fn = static_cast<int64_t>(fnx) * fny * fnz;
    const int32_t ix = I % cnx, iy = (I / cnx) % cny, iz = I / (cnx * cny);
    // cells of the block per direction (1 at the end of an odd side)
    const int32_t sx = fnx - 2 * ix < 2 ? 1 : 2, sy = fny - 2 * iy < 2 ? 1 : 2, sz = fnz - 2 * iz < 2 ? 1 : 2;
    double dg = 0.0;
    for (int e = 0; e < sz; ++e)
        for (int bb = 0; bb < sy; ++bb)
            for (int a = 0; a < sx; ++a)
                dg += diag[(2 * ix + a) + fnx * ((2 * iy + bb) + fny * (2 * iz + e))];
    for (int e = 0; e < sz; ++e)
        for (int bb = 0; bb < sy; ++bb)
            for (int a = 0; a < sx; ++a) {
                const int64_t c = (2 * ix + a) + fnx * ((2 * iy + bb) + static_cast<int64_t>(fny) * (2 * iz + e));
                if (a + 1 < sx) dg += 2.0 * coef[c];
                if (bb + 1 < sy) dg += 2.0 * coef[fn + c];
                if (e + 1 < sz) dg += 2.0 * coef[2 * fn + c];
            }
    cdiag[I] = dg;
    // the crossing faces in each direction
    const int32_t span[3] = {sx, sy, sz};
    for (int k = 0; k < 3; ++k) {
        double u = 0.0;
        if (span[k] == 2) {
            for (int e = 0; e < sz; ++e)
                for (int bb = 0; bb < sy; ++bb)
                    for (int a = 0; a < sx; ++a) {
                        const int side = k == 0 ? a : (k == 1 ? bb : e);
                        if (side != 1) continue;
                        const int64_t c =
                            (2 * ix + a) + fnx * ((2 * iy + bb) + static_cast<int64_t>(fny) * (2 * iz + e));
                        u += coef[k * fn + c];
                    }
        }
        ccoef[static_cast<int64_t>(k) * cn + I] = u;
    }
}

// the block walk of each level (index 0: the problem's own box) where its
// x-lines have even length, and whether its sides are all even (then the
// restriction to the next level runs on it too)
static void plan_amg_walks(lf_problem *P) {
    const lf_mesh *m = P->mesh;
    const size_t nl = P->amg.size() + 1;
    P->amg_bw.assign(nl, BoxWalk{});
    P->amg_walk.assign(nl, 0);
    for (size_t l = 0; l < nl; ++l) {
        const int32_t nx = l == 0 ? m->box_nx : P->amg[l - 1].nx, ny = l == 0 ? m->box_ny : P->amg[l - 1].ny;
        const int32_t nz = l == 0 ? m->box_nz : P->amg[l - 1].nz;
        const int32_t d[3] = {1, nx, nx * ny};
        BoxWalk bw;
        // LF_WALK_ON takes it on every level that allows it (tests), LF_WALK_OFF on none
        const int32_t wo = P->opts.amul_walk;
        if (wo != LF_WALK_OFF && nx % 2 == 0 && box_walk_plan(nx * ny * nz, 3, d, 2, &bw) &&
            (wo == LF_WALK_ON || bw.blocks >= kAmgWalkMinBlocks) && bw.blocks <= P->sp.grid) {
            P->amg_bw[l] = bw;
            P->amg_walk[l] = (ny % 2 == 0 && nz % 2 == 0) ? 2 : 1;
        }
    }
}

// the first level whose cycle runs in one workgroup (0: none).  LF_WALK_ON
// keeps the launches, so that the walk runs on every level that allows it.
static void plan_amg_tail(lf_problem *P) {
    const size_t levels = P->amg.size() + 1;
    int64_t rows = 0;
    size_t first = 0;
    for (size_t l = levels; l-- > 1 && levels - l <= static_cast<size_t>(kTailLevels);) {
        rows += P->amg[l - 1].n;
        if (rows > kTailRows) break;
        first = l;
    }
    P->amg_tail = 0;
    if (first == 0 || P->opts.amul_walk == LF_WALK_ON) return;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(&k_amg_tail), hipFuncAttributeMaxDynamicSharedMemorySize,
                            156 << 10) == hipSuccess)
        P->amg_tail = first;
    else
        (void)hipGetLastError();
}

static dim3 grid_for(int64_t n) {
    return dim3(static_cast<unsigned>(std::max<int64_t>(1, (n + kCellBlock - 1) / kCellBlock)));
}

// the matrix, right side and work vectors of level l (0: the problem's own)
struct AmgView {
    int32_t nx, ny, nz;
    const double *coef, *diag;
    double *ta, *tb;
};

static AmgView amg_view(const lf_problem *P, size_t l) {
    const lf_mesh *m = P->mesh;
    if (l == 0) return AmgView{m->box_nx, m->box_ny, m->box_nz, P->coef, P->diagB, P->amg_t1, P->amg_t2};
    const AmgLevel &a = P->amg[l - 1];
    return AmgView{a.nx, a.ny, a.nz, a.coef, a.diag, a.xa, a.xb};
}

void launch_amg_galerkin(lf_problem *P, hipStream_t s) {
    for (size_t l = 1; l <= P->amg.size(); ++l) {
        const AmgView f = amg_view(P, l - 1);
        const AmgLevel &c = P->amg[l - 1];
        LF_LAUNCH(P, LF_K_AMG_GALERKIN, s, k_amg_galerkin, grid_for(c.n), dim3(kCellBlock), 0, s, f.nx, f.ny, f.nz,
                  f.diag, f.coef, c.nx, c.ny, c.nz, c.diag, c.coef);
    }
}

static const double *amg_tail(lf_problem *P, size_t l, const double *b, hipStream_t s) {
    AmgTail T{};
    int32_t rows = 0;
    for (size_t k = l; k <= P->amg.size(); ++k) {
        const AmgLevel &a = P->amg[k - 1];
        const int32_t i = T.count++;
        T.nx[i] = a.nx;
        T.ny[i] = a.ny;
        T.nz[i] = a.nz;
        T.off[i] = rows;
        T.coef[i] = a.coef;
        T.diag[i] = a.diag;
        rows += a.n;
    }
    T.b = b;
    T.x = P->amg[l - 1].xa;
    const size_t lds = 7 * sizeof(double) * static_cast<size_t>(rows);
    LF_LAUNCH(P, LF_K_AMG_SMOOTH, s, k_amg_tail, dim3(1), dim3(kTailBlock), static_cast<unsigned>(lds), s, T,
              P->state);
    return T.x;
}

// One sweep of level v into dst, x from the source, by the block walk where the
// level has one; dot: with the w.r partials (level 0's last sweep).
template <class XS>
static void launch_sweep(lf_problem *P, const AmgView &v, const BandLayout<3> &L, bool walk, const BoxWalk &bw,
                         const double *b, const XS &x, double *dst, bool dot, hipStream_t s) {
    if (walk) {
        const dim3 grid(static_cast<unsigned>(std::max<int32_t>(1, bw.blocks)));
        if (dot)
            LF_LAUNCH(P, LF_K_AMG_SMOOTH, s, (k_amg_sweep_box<XS, true>), grid, dim3(kBwBlock), 0, s, P->sp, L, bw,
                      v.diag, v.coef, b, x, dst, P->part, P->state);
        else
            LF_LAUNCH(P, LF_K_AMG_SMOOTH, s, (k_amg_sweep_box<XS, false>), grid, dim3(kBwBlock), 0, s, P->sp, L, bw,
                      v.diag, v.coef, b, x, dst, P->part, P->state);
    } else {
        if (dot)
            LF_LAUNCH(P, LF_K_AMG_SMOOTH, s, (k_amg_sweep<XS, true>), grid_for(L.n), dim3(kCellBlock), 0, s, P->sp, L,
                      v.diag, v.coef, b, x, dst, P->part, P->state);
        else
            LF_LAUNCH(P, LF_K_AMG_SMOOTH, s, (k_amg_sweep<XS, false>), grid_for(L.n), dim3(kCellBlock), 0, s, P->sp,
                      L, v.diag, v.coef, b, x, dst, P->part, P->state);
    }
}

// One cycle on level l for the right side b; the result ends in `out` when
// given (level 0: w, with the w.r partials), else in one of the level's work
// vectors, which is returned.  The first two sweeps are one launch, and the
// first sweep after the coarse correction also adds it.
static const double *amg_cycle(lf_problem *P, size_t l, const double *b, double *out, hipStream_t s) {
    if (l > 0 && l == P->amg_tail) return amg_tail(P, l, b, s);
    const AmgView v = amg_view(P, l);
    const BandLayout<3> L = box_layout(v.nx, v.ny, v.nz);
    const bool coarsest = l == P->amg.size();
    const int walk = P->amg_walk[l];
    const BoxWalk bw = P->amg_bw[l];
    typedef MemX<double, 2> X;
    launch_sweep(P, v, L, walk, bw, b, AmgFirstX{b, v.diag}, v.ta, false, s);
    if (coarsest) {
        launch_sweep(P, v, L, walk, bw, b, X{v.ta}, v.tb, false, s);
        double *dst = out ? out : v.ta;
        launch_sweep(P, v, L, walk, bw, b, X{v.tb}, dst, l == 0, s);
        return dst;
    }
    AmgLevel &c = P->amg[l];
    if (walk == 2)
        LF_LAUNCH(P, LF_K_AMG_RESTRICT, s, k_amg_restrict_box, dim3(static_cast<unsigned>(bw.blocks)), dim3(kBwBlock),
                  0, s, L, bw, v.diag, v.coef, b, v.ta, c.b, P->state);
    else
        LF_LAUNCH(P, LF_K_AMG_RESTRICT, s, k_amg_restrict, grid_for(8 * static_cast<int64_t>(c.n)),
                  dim3(kCellBlock), 0, s, L, v.nx, v.ny, v.nz, v.diag, v.coef, b, v.ta, c.nx, c.ny, c.n, c.b, P->state);
    const double *xc = amg_cycle(P, l + 1, c.b, nullptr, s);
    const AmgProlongX px{v.ta, xc, v.nx, v.ny, c.nx, c.ny, fast_div(static_cast<uint32_t>(v.nx)),
                         fast_div(static_cast<uint32_t>(v.ny))};
    launch_sweep(P, v, L, walk, bw, b, px, v.tb, false, s);
    double *dst = out ? out : v.ta;
    launch_sweep(P, v, L, walk, bw, b, X{v.tb}, dst, l == 0, s);
    return dst;
}

void launch_amg_cycle(lf_problem *P, hipStream_t s) { amg_cycle(P, 0, P->r, P->w, s); }

}  // namespace lf
