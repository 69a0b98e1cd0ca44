// Kernels of the mesh step around the interface estimate (FP64):
//   * edge_gen_kernel: the one-dimensional form of the generator (eq. Gen,
//     section 2) along each physical side, which gives the tangential
//     boundary values at t^{n+1};
//   * targets_kernel: Dirichlet data of the decomposed problem at t^{n+1}
//     (physical boundary, interface estimate, images of the seam);
//   * subdomain_lds_kernel: the subdomain solves of section 3.5 (centred
//     differences, forward Euler), one workgroup per subdomain with the
//     subdomain's mesh resident in LDS for all substeps;
//   * fe_tile_kernel: several forward-Euler substeps over the whole grid in
//     one launch, tile by tile in LDS; used when a subdomain does not fit one
//     workgroup and for the single-domain reference (periodic axes wrap);
//   * fe_sweep_kernel: one substep over the whole grid in global memory, the
//     first of a periodic single domain (it reads the image nodes as given);
//   * arclength kernels: the monitor rho = sqrt(1 + a |grad u|^2) from nodal u
//     on the new mesh (section 3.6), the physical gradient through the
//     inverse mesh Jacobian;
//   * quality kernels: Q(K) per cell (eq. Q, section 3.7) of two meshes, the
//     ratio R = Q_SD / Q_SDD, its maximum and its mean (fixed-order sums).
//
// Floating-point contraction is off in this file: every update is the plain
// sequence of IEEE operations written below, in that order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "msdd_mesh_step.hpp"

#pragma clang fp contract(off)

namespace msdd {

namespace {

__device__ __forceinline__ int side_offset(int side, int comp, int n_xi, int n_eta)
{
    return side < 2 ? (side * 2 + comp) * n_eta : 4 * n_eta + ((side - 2) * 2 + comp) * n_xi;
}

// ---------------------------------------------------------------------------
// 1-D generator along the physical sides
// ---------------------------------------------------------------------------
// Workgroup k advances one side: sides 0, 1 (xi = 0, 1; y runs along eta)
// when xi is a Dirichlet axis, sides 2, 3 (eta = 0, 1; x runs along xi)
// when eta is.  LDS holds the two time levels and the drift coefficients.
// P2: n - 1 is a power of two on every side, so the divisors h are, and the
// divisions go into the coefficients exactly (as in fe_update).  Bound: the
// chain of one substep (LDS read, update, LDS write, barrier), so one node
// per thread up to 1024: 129 nodes, 1457 substeps 104 -> 51 us; 257 nodes,
// periodic, 728 substeps 380 -> 175 us (256 threads took the last node in a
// second round).
template <bool P2>
__global__ __launch_bounds__(kEdgeBlock) void edge_gen_kernel(const double *__restrict__ rho,
                                                             const double *__restrict__ rho_xi,
                                                             const double *__restrict__ rho_eta, int n_xi,
                                                             int n_eta, int per_xi, int per_eta, double Lx,
                                                             double Ly, double tau, int L_eta, int L_xi,
                                                             double *__restrict__ bnd)
{
    extern __shared__ double sm[];
    const int side = per_xi ? (int)blockIdx.x + 2 : (int)blockIdx.x;
    const bool along_eta = side < 2;
    const int n = along_eta ? n_eta : n_xi;
    const int L = along_eta ? L_eta : L_xi;
    const int periodic = along_eta ? per_eta : per_xi;
    const double period = along_eta ? Ly : Lx;
    const int off = side_offset(side, along_eta ? 1 : 0, n_xi, n_eta);
    double *cur = sm, *nxt = sm + n, *bb = sm + 2 * n;
    const double h = 1.0 / (double)(n - 1);
    const double two_h = 2.0 * h, hh = h * h;
    const double scale = P2 ? hh / two_h : 1.0;
    const double dt = P2 ? tau / (double)L / hh : tau / (double)L;
    for (int s = threadIdx.x; s < n; s += blockDim.x) {
        const int g = along_eta ? s * n_xi + (side == 0 ? 0 : n_xi - 1) : (side == 2 ? 0 : n_eta - 1) * n_xi + s;
        cur[s] = bnd[off + s];
        bb[s] = (along_eta ? rho_eta[g] : rho_xi[g]) / rho[g] * scale;
    }
    __syncthreads();
    auto update = [&](double b, double c, double left, double right) {
        if (P2) return c + dt * (b * (right - left) + (__builtin_fma(-2.0, c, right) + left));
        return c + dt * (b * (right - left) / two_h + (right - 2.0 * c + left) / hh);
    };
    // the value of node s one substep on; node n-1 of a periodic side is the
    // image of node 0: its update is node 0's plus the period
    auto next = [&](int s, double b, double c) {
        if (periodic) {
            const bool image = s == n - 1;
            const int q = image ? 0 : s;
            const double left = q > 0 ? cur[q - 1] : cur[n - 2] - period;
            const double v = update(b, image ? cur[0] : c, left, cur[q + 1]);
            return image ? v + period : v;
        }
        return s == 0 || s == n - 1 ? c : update(b, c, cur[s - 1], cur[s + 1]);
    };
    if (n <= (int)blockDim.x) {   // one node per thread, its value and coefficient in registers
        const int s = threadIdx.x;
        double c = s < n ? cur[s] : 0.0;
        const double b = s < n ? bb[periodic && s == n - 1 ? 0 : s] : 0.0;
        for (int l = 0; l < L; ++l) {
            if (s < n) {
                c = next(s, b, c);
                nxt[s] = c;
            }
            __syncthreads();
            double *t = cur;
            cur = nxt;
            nxt = t;
        }
    } else {
        for (int l = 0; l < L; ++l) {
            for (int s = threadIdx.x; s < n; s += blockDim.x)
                nxt[s] = next(s, bb[periodic && s == n - 1 ? 0 : s], cur[s]);
            __syncthreads();
            double *t = cur;
            cur = nxt;
            nxt = t;
        }
    }
    for (int s = threadIdx.x; s < n; s += blockDim.x) bnd[off + s] = cur[s];
}

// ---------------------------------------------------------------------------
// Dirichlet data at t^{n+1}
// ---------------------------------------------------------------------------
struct Target {
    double x, y;
    bool dirichlet;
};

__device__ Target target_of(int i, int j, const MeshStepArgs &a)
{
    // with interfaces, an image node on a periodic axis follows its original
    double ox = 0.0, oy = 0.0;
    if (a.with_interfaces) {
        if (a.per_xi && i == a.n_xi - 1) {
            i = 0;
            ox = a.Lx;
        }
        if (a.per_eta && j == a.n_eta - 1) {
            j = 0;
            oy = a.Ly;
        }
    }
    Target t{0.0, 0.0, false};
    if (a.with_interfaces) {
        const int r = a.node_rank[j * a.n_xi + i];
        if (r >= 0) t = Target{a.iface_x[r], a.iface_y[r], true};
    }
    if (!a.per_xi && (i == 0 || i == a.n_xi - 1)) {
        const int side = i == 0 ? 0 : 1;
        t = Target{a.bnd1[side_offset(side, 0, a.n_xi, a.n_eta) + j], a.bnd1[side_offset(side, 1, a.n_xi, a.n_eta) + j],
                   true};
    }
    if (!a.per_eta && (j == 0 || j == a.n_eta - 1)) {   // rows win at corners
        const int side = j == 0 ? 2 : 3;
        t = Target{a.bnd1[side_offset(side, 0, a.n_xi, a.n_eta) + i], a.bnd1[side_offset(side, 1, a.n_xi, a.n_eta) + i],
                   true};
    }
    t.x = t.x + ox;
    t.y = t.y + oy;
    return t;
}

__global__ void targets_kernel(MeshStepArgs a, double *__restrict__ x_new, double *__restrict__ y_new)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= a.n_xi * a.n_eta) return;
    const int i = g % a.n_xi, j = g / a.n_xi;
    const Target t = target_of(i, j, a);
    a.mask[g] = t.dirichlet ? 1 : 0;
    // the drift coefficients of a node that is advanced take the place of its
    // Dirichlet values, so no launch of the solve divides again
    a.tx1[g] = t.dirichlet ? t.x : a.rho_xi[g] / a.rho[g];
    a.ty1[g] = t.dirichlet ? t.y : a.rho_eta[g] / a.rho[g];
    if (t.dirichlet) {
        x_new[g] = t.x;
        y_new[g] = t.y;
    }
}

// ---------------------------------------------------------------------------
// The forward-Euler update
// ---------------------------------------------------------------------------
// One substep of a node, with the roundings of the plain expression
//   c + dt (bx (e - w) / 2hx + by (n - s) / 2hy + (e - 2c + w) / hx^2 + (n - 2c + s) / hy^2).
// P2: the cell counts of both axes are powers of two.  Every divisor is then a
// power of two, which scales exactly, so the whole sum is taken in units of
// 1 / hx^2 and the divisions go into bx, by and dt (13 operations and one for
// hy != hx instead of 17 and four divisions); e - 2c is one rounding either
// way.  Otherwise the divisions stay: bx, by are the plain coefficients.
struct FeCoef {
    double two_hx, two_hy, hxx, hyy, dt;   // P2: dt / hx^2 in dt, hx^2 / hy^2 in hyy
    double sx, sy;                         // P2: scales of bx and by
};

template <bool P2>
__device__ __forceinline__ FeCoef fe_coef(const MeshStepArgs &a)
{
    const double hx = 1.0 / (double)(a.n_xi - 1), hy = 1.0 / (double)(a.n_eta - 1);
    FeCoef k;
    k.two_hx = 2.0 * hx;
    k.two_hy = 2.0 * hy;
    k.hxx = hx * hx;
    k.hyy = hy * hy;
    k.dt = a.tau / (double)a.L;
    k.sx = k.sy = 1.0;
    if (P2) {
        k.sx = k.hxx / k.two_hx;
        k.sy = k.hxx / k.two_hy;
        k.hyy = k.hxx / k.hyy;
        k.dt = k.dt / k.hxx;
    }
    return k;
}

template <bool P2>
__device__ __forceinline__ double fe_update(const FeCoef &k, double bx, double by, double c, double e, double w,
                                            double n, double s)
{
    if (P2)
        return c + k.dt * (bx * (e - w) + by * (n - s) + (__builtin_fma(-2.0, c, e) + w) +
                           (__builtin_fma(-2.0, c, n) + s) * k.hyy);
    return c + k.dt * (bx * (e - w) / k.two_hx + by * (n - s) / k.two_hy + (e - 2.0 * c + w) / k.hxx +
                       (n - 2.0 * c + s) / k.hyy);
}

// ---------------------------------------------------------------------------
// Subdomain solves with the subdomain resident in LDS
// ---------------------------------------------------------------------------
// One workgroup per subdomain, all substeps in one launch, two time levels in
// LDS, one barrier per substep.  Without divisions (P2) a thread owns R nodes
// of a column (its north and south neighbours then are its own registers but
// for two), the last segment of a column overlapping the one before it; with
// them it owns the nodes t, t + inner, ... of the box.  The threads from
// `first_bnd` on own a boundary node each (beside their other nodes where the
// workgroup is full).  Bound: LDS reads and FP64 issue of one CU (33x33 box
// without divisions: 5 + 2 LDS values and 28 operations per node and
// substep, about 420 clocks of each), then the barrier.  16 boxes of 33x33,
// 729 substeps: 1.10 ms with a node per thread, four divisions per update and
// two barriers, 0.34 ms now.
template <bool P2, int R>
__global__ __launch_bounds__(kSubBlock) void subdomain_lds_kernel(MeshStepArgs a, int inner, int first_bnd,
                                                                  double *__restrict__ x_new,
                                                                  double *__restrict__ y_new)
{
    extern __shared__ double sm[];
    const int bi = (int)blockIdx.x % a.sub_xi, bj = (int)blockIdx.x / a.sub_xi;
    const int Px = a.P_xi, Py = a.P_eta;
    const int Bx = Px + 1, By = Py + 1, n = Bx * By;
    const int i0 = bi * Px, j0 = bj * Py;
    double *cur = sm, *nxt = sm + 2 * n;   // x, then y, of each level
    const int tid = threadIdx.x;
    for (int q = tid; q < n; q += blockDim.x) {
        const int g = (j0 + q / Bx) * a.n_xi + i0 + q % Bx;
        cur[q] = a.x0[g];
        cur[n + q] = a.y0[g];
    }
    const FeCoef k = fe_coef<P2>(a);
    // own interior nodes, -1: none; q[r] = q[0] + r Bx in a segment (and one
    // node is a segment of one)
    constexpr bool kSegment = P2 || R == 1;
    const int segs = (Px - 1) * ((Py - 1 + R - 1) / R), nin = (Px - 1) * (Py - 1);
    int q[R], qb = 0;   // and the boundary node
    double bx[R], by[R], x[R], y[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int k1 = kSegment ? tid : tid + r * inner;
        q[r] = -1;
        if (tid < inner && k1 < (kSegment ? segs : nin)) {
            const int ca = 1 + k1 % (Px - 1), row = k1 / (Px - 1);
            const int cc = kSegment ? min(1 + row * R, Py - R) + r : 1 + row;
            const int g = (j0 + cc) * a.n_xi + i0 + ca;
            q[r] = cc * Bx + ca;
            bx[r] = a.tx1[g] * k.sx;
            by[r] = a.ty1[g] * k.sy;
            x[r] = a.x0[g];
            y[r] = a.y0[g];
        }
    }
    const int nb = 2 * Bx + 2 * (By - 2);
    const int tb = tid - first_bnd;
    const bool edge = tb >= 0 && tb < nb;
    double bx0 = 0.0, by0 = 0.0, bx1 = 0.0, by1 = 0.0;
    if (edge) {
        int ca, cc;
        if (tb < Bx) {
            ca = tb;
            cc = 0;
        } else if (tb < 2 * Bx) {
            ca = tb - Bx;
            cc = By - 1;
        } else if (tb < 2 * Bx + By - 2) {
            ca = 0;
            cc = 1 + tb - 2 * Bx;
        } else {
            ca = Bx - 1;
            cc = 1 + tb - 2 * Bx - (By - 2);
        }
        const int g = (j0 + cc) * a.n_xi + i0 + ca;
        qb = cc * Bx + ca;
        bx0 = a.x0[g];
        by0 = a.y0[g];
        bx1 = a.tx1[g];
        by1 = a.ty1[g];
    }
    __syncthreads();
    for (int l = 0; l < a.L; ++l) {
        if (kSegment && q[0] >= 0) {
            const double *px = cur + q[0], *py = px + n;
            double e[R], w[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                e[r] = px[r * Bx + 1];
                w[r] = px[r * Bx - 1];
            }
            double below = px[-Bx];
            const double above = px[R * Bx];
            double e2[R], w2[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                e2[r] = py[r * Bx + 1];
                w2[r] = py[r * Bx - 1];
            }
            double below2 = py[-Bx];
            const double above2 = py[R * Bx];
            double *ox = nxt + q[0], *oy = ox + n;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double v = fe_update<P2>(k, bx[r], by[r], x[r], e[r], w[r], r + 1 < R ? x[r + 1] : above, below);
                below = x[r];
                x[r] = v;
                ox[r * Bx] = v;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double v =
                    fe_update<P2>(k, bx[r], by[r], y[r], e2[r], w2[r], r + 1 < R ? y[r + 1] : above2, below2);
                below2 = y[r];
                y[r] = v;
                oy[r * Bx] = v;
            }
        }
        if (!kSegment) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (q[r] >= 0) {
                    const double *px = cur + q[r], *py = px + n;
                    x[r] = fe_update<P2>(k, bx[r], by[r], x[r], px[1], px[-1], px[Bx], px[-Bx]);
                    y[r] = fe_update<P2>(k, bx[r], by[r], y[r], py[1], py[-1], py[Bx], py[-Bx]);
                    nxt[q[r]] = x[r];
                    nxt[n + q[r]] = y[r];
                }
        }
        if (edge) {
            const double th1 = (double)(l + 1) / (double)a.L;
            nxt[qb] = (1.0 - th1) * bx0 + th1 * bx1;
            nxt[n + qb] = (1.0 - th1) * by0 + th1 * by1;
        }
        __syncthreads();
        double *t = cur;
        cur = nxt;
        nxt = t;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (q[r] >= 0) {
            const int g = (j0 + q[r] / Bx) * a.n_xi + i0 + q[r] % Bx;
            x_new[g] = x[r];
            y_new[g] = y[r];
        }
}

// ---------------------------------------------------------------------------
// Several substeps of the whole grid in one launch
// ---------------------------------------------------------------------------
// For boxes (subdomains, or the single domain) that one workgroup does not
// hold.  A workgroup advances a tile of kTileCore^2 nodes by a.steps substeps
// in LDS, with a rim of kTileRim nodes on each side, of which each substep
// uses up one: the nodes of the rim are computed again by the neighbours,
// and no workgroup waits for another.  Beyond a Dirichlet side of the box
// there is nothing to compute, so the rim ends there; Dirichlet nodes follow
// their line in time by themselves.  On a periodic axis (PER; the single
// domain) the rim goes round: nodes are held by their index 0 .. n-2, and a
// neighbour across the seam is the node there plus or minus the period, the
// rounding of which is that of the stored image.
// A thread owns kTileRows nodes of a column.  Bound: the launch and the loads
// of a tile (about 5 us) and the FP64 issue of its 32 x 32 nodes (0.4 us a
// substep).  Cores of 16 with a rim of 8 and two rows per thread, on 257^2:
// rims of 6, 12, 16 and cores of 24 are 15 to 40 % slower, four rows 8 %.  257^2,
// 1457 substeps: 1457 sweeps 5.1 ms, 182 tile launches 1.6 ms.
template <bool P2, bool PER>
__global__ __launch_bounds__(kTileSide *kTileSide / kTileRows) void fe_tile_kernel(
    MeshStepArgs a, const double *__restrict__ cx, const double *__restrict__ cy, double *__restrict__ nx,
    double *__restrict__ ny)
{
    constexpr int S = kTileSide, R = kTileRows;
    // one row and one node more on each side, read by the outermost threads
    // only and never part of a result
    __shared__ double sm[2][2][(S + 2) * S + 2];
    const bool pxi = PER && a.per_xi, peta = PER && a.per_eta;
    // nodes of a box that are advanced: the inner ones, all distinct ones along a periodic axis
    const int nix = pxi ? a.n_xi - 1 : a.P_xi - 1, niy = peta ? a.n_eta - 1 : a.P_eta - 1;
    const int tiles_x = (nix + kTileCore - 1) / kTileCore, tiles_y = (niy + kTileCore - 1) / kTileCore;
    const int box = (int)blockIdx.x / (tiles_x * tiles_y), tile = (int)blockIdx.x % (tiles_x * tiles_y);
    const int bi = box % a.sub_xi, bj = box / a.sub_xi;
    const int ox = bi * a.P_xi + (pxi ? 0 : 1) + tile % tiles_x * kTileCore;   // first node of the core
    const int oy = bj * a.P_eta + (peta ? 0 : 1) + tile / tiles_x * kTileCore;
    const int lo_x = bi * a.P_xi, hi_x = lo_x + a.P_xi, lo_y = bj * a.P_eta, hi_y = lo_y + a.P_eta;
    const int col = threadIdx.x % S, row0 = (int)threadIdx.x / S * R;
    const FeCoef k = fe_coef<P2>(a);

    // own nodes: 0 outside the box, 1 Dirichlet, 2 advanced
    int kind[R], gi[R];
    double p0[R], p1[R], p2[R], p3[R], x[R], y[R], eo = 0.0, wo = 0.0, no[R], so[R];
    int i = ox - kTileRim + col;
    bool in_x = pxi || (i >= lo_x && i <= hi_x), edge_x = !pxi && (i == lo_x || i == hi_x);
    if (pxi) {
        const int m = a.n_xi - 1;
        i = ((i % m) + m) % m;
        eo = i == m - 1 ? a.Lx : 0.0;
        wo = i == 0 ? 0.0 - a.Lx : 0.0;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int j = oy - kTileRim + row0 + r;
        const bool in_y = peta || (j >= lo_y && j <= hi_y), edge_y = !peta && (j == lo_y || j == hi_y);
        no[r] = so[r] = 0.0;
        if (peta) {
            const int m = a.n_eta - 1;
            j = ((j % m) + m) % m;
            no[r] = j == m - 1 ? a.Ly : 0.0;
            so[r] = j == 0 ? 0.0 - a.Ly : 0.0;
        }
        kind[r] = !(in_x && in_y) ? 0 : (edge_x || edge_y) ? 1 : 2;
        const int g = kind[r] ? j * a.n_xi + i : 0;
        gi[r] = g;
        x[r] = y[r] = p0[r] = p1[r] = p2[r] = p3[r] = 0.0;
        if (kind[r] == 2) {
            x[r] = cx[g];
            y[r] = cy[g];
            p0[r] = a.tx1[g] * k.sx;
            p1[r] = a.ty1[g] * k.sy;
        } else if (kind[r] == 1) {
            p0[r] = a.x0[g];
            p1[r] = a.tx1[g];
            p2[r] = a.y0[g];
            p3[r] = a.ty1[g];
            const double th = (double)a.l0 / (double)a.L;
            x[r] = a.l0 == 0 ? p0[r] : (1.0 - th) * p0[r] + th * p1[r];
            y[r] = a.l0 == 0 ? p2[r] : (1.0 - th) * p2[r] + th * p3[r];
        }
    }
    const int q0 = (row0 + 1) * S + col + 1;
    bool edge = false, seam = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        sm[0][0][q0 + r * S] = x[r];
        sm[0][1][q0 + r * S] = y[r];
        edge = edge || kind[r] == 1;
        if (PER) seam = seam || no[r] != 0.0 || so[r] != 0.0;
    }
    if (PER) seam = seam || eo != 0.0 || wo != 0.0;
    // most waves hold no Dirichlet node and no node beside a seam
    const bool any_edge = __ballot(edge) != 0, any_seam = PER && __ballot(seam) != 0;
    __syncthreads();
    for (int l = 0; l < a.steps; ++l) {
        const double *px = &sm[l & 1][0][q0], *py = &sm[l & 1][1][q0];
        double *qx = &sm[(l & 1) ^ 1][0][q0], *qy = &sm[(l & 1) ^ 1][1][q0];
        double bel = px[-S], bel2 = py[-S];
        const double abv = px[R * S], abv2 = py[R * S];
        double e[R], w[R], e2[R], w2[R], n2[R], s2[R], u[R], v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            e[r] = px[r * S + 1];
            w[r] = px[r * S - 1];
            e2[r] = py[r * S + 1];
            w2[r] = py[r * S - 1];
            n2[r] = r + 1 < R ? y[r + 1] : abv2;
            s2[r] = r > 0 ? y[r - 1] : bel2;
        }
        if (any_seam) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                e[r] = e[r] + eo;
                w[r] = w[r] + wo;
                n2[r] = n2[r] + no[r];
                s2[r] = s2[r] + so[r];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            u[r] = fe_update<P2>(k, p0[r], p1[r], x[r], e[r], w[r], r + 1 < R ? x[r + 1] : abv, r > 0 ? x[r - 1] : bel);
            v[r] = fe_update<P2>(k, p0[r], p1[r], y[r], e2[r], w2[r], n2[r], s2[r]);
        }
        if (any_edge) {
            const double th1 = (double)(a.l0 + l + 1) / (double)a.L;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (kind[r] == 1) {
                    u[r] = (1.0 - th1) * p0[r] + th1 * p1[r];
                    v[r] = (1.0 - th1) * p2[r] + th1 * p3[r];
                }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            x[r] = u[r];
            y[r] = v[r];
            qx[r * S] = u[r];
            qy[r * S] = v[r];
        }
        __syncthreads();
    }
    // the core's advanced nodes, and the images of node 0 on a periodic axis
    const int c = col - kTileRim;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int d = row0 + r - kTileRim;
        if (kind[r] != 2 || c < 0 || c >= kTileCore || d < 0 || d >= kTileCore) continue;
        if (PER && ((pxi && ox + c > a.n_xi - 2) || (peta && oy + d > a.n_eta - 2))) continue;   // gone round
        const int g = gi[r];
        nx[g] = x[r];
        ny[g] = y[r];
        if (PER) {
            const int ii = g % a.n_xi, jj = g / a.n_xi;
            const bool ix = pxi && ii == 0, iy = peta && jj == 0;
            const int gx = jj * a.n_xi + a.n_xi - 1, gy = (a.n_eta - 1) * a.n_xi + ii;
            if (ix) nx[gx] = x[r] + a.Lx, ny[gx] = y[r];
            if (iy) nx[gy] = x[r], ny[gy] = y[r] + a.Ly;
            if (ix && iy) {
                const int gc = a.n_eta * a.n_xi - 1;
                nx[gc] = x[r] + a.Lx;
                ny[gc] = y[r] + a.Ly;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// One forward-Euler substep over the whole grid in global memory
// ---------------------------------------------------------------------------
__device__ __forceinline__ double nb_value(const double *f, int i, int j, const MeshStepArgs &a, double L_xi,
                                           double L_eta)
{
    double off = 0.0;
    if (a.per_xi) {
        if (i < 0) {
            i += a.n_xi - 1;
            off -= L_xi;
        } else if (i > a.n_xi - 1) {
            i -= a.n_xi - 1;
            off += L_xi;
        }
    }
    if (a.per_eta) {
        if (j < 0) {
            j += a.n_eta - 1;
            off -= L_eta;
        } else if (j > a.n_eta - 1) {
            j -= a.n_eta - 1;
            off += L_eta;
        }
    }
    return f[j * a.n_xi + i] + off;
}

__device__ __forceinline__ double stencil(const double *f, int i, int j, const MeshStepArgs &a, double L_xi,
                                          double L_eta, double bx, double by, double dt, double two_hx,
                                          double two_hy, double hxx, double hyy)
{
    const double c = f[j * a.n_xi + i];
    const double e = nb_value(f, i + 1, j, a, L_xi, L_eta), w = nb_value(f, i - 1, j, a, L_xi, L_eta);
    const double n = nb_value(f, i, j + 1, a, L_xi, L_eta), s = nb_value(f, i, j - 1, a, L_xi, L_eta);
    return c + dt * (bx * (e - w) / two_hx + by * (n - s) / two_hy + (e - 2.0 * c + w) / hxx + (n - 2.0 * c + s) / hyy);
}

__global__ void fe_sweep_kernel(MeshStepArgs a, const double *__restrict__ cx, const double *__restrict__ cy,
                                double *__restrict__ nx, double *__restrict__ ny, double th1)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= a.n_xi * a.n_eta) return;
    if (a.mask[g]) {
        nx[g] = (1.0 - th1) * a.x0[g] + th1 * a.tx1[g];
        ny[g] = (1.0 - th1) * a.y0[g] + th1 * a.ty1[g];
        return;
    }
    int i = g % a.n_xi, j = g / a.n_xi;
    // an image node (periodic axis, not Dirichlet) repeats its original's update plus the period
    double ox = 0.0, oy = 0.0;
    if (a.per_xi && i == a.n_xi - 1) {
        i = 0;
        ox = a.Lx;
    }
    if (a.per_eta && j == a.n_eta - 1) {
        j = 0;
        oy = a.Ly;
    }
    const int s = j * a.n_xi + i;
    const double hx = 1.0 / (double)(a.n_xi - 1), hy = 1.0 / (double)(a.n_eta - 1);
    const double bx = a.rho_xi[s] / a.rho[s], by = a.rho_eta[s] / a.rho[s];
    const double dt = a.tau / (double)a.L;
    const double vx = stencil(cx, i, j, a, a.Lx, 0.0, bx, by, dt, 2.0 * hx, 2.0 * hy, hx * hx, hy * hy);
    const double vy = stencil(cy, i, j, a, 0.0, a.Ly, bx, by, dt, 2.0 * hx, 2.0 * hy, hx * hx, hy * hy);
    nx[g] = ox != 0.0 ? vx + ox : vx;
    ny[g] = oy != 0.0 ? vy + oy : vy;
}

// ---------------------------------------------------------------------------
// Arc-length monitor from nodal u
// ---------------------------------------------------------------------------
// Difference along one axis in units of the node index: centred inside,
// one-sided second order at Dirichlet ends, wrapped (plus `period` for the
// winding coordinate) on a periodic axis.  `stride` steps along the axis.
__device__ __forceinline__ double axis_diff(const double *f, int base, int k, int n, int stride, int periodic,
                                            double period)
{
    if (periodic) {
        double left, right;
        if (k == 0 || k == n - 1) {
            left = f[base + (n - 2) * stride] - period;
            right = f[base + stride];
        } else {
            left = f[base + (k - 1) * stride];
            right = f[base + (k + 1) * stride];
        }
        return 0.5 * (right - left);
    }
    if (k == 0) return 0.5 * (-3.0 * f[base] + 4.0 * f[base + stride] - f[base + 2 * stride]);
    if (k == n - 1)
        return 0.5 * (3.0 * f[base + (n - 1) * stride] - 4.0 * f[base + (n - 2) * stride] + f[base + (n - 3) * stride]);
    return 0.5 * (f[base + (k + 1) * stride] - f[base + (k - 1) * stride]);
}

__global__ void arclength_grad_kernel(const double *__restrict__ u, const double *__restrict__ x,
                                      const double *__restrict__ y, int n_xi, int n_eta, int per_xi, int per_eta,
                                      double Lx, double Ly, double *__restrict__ g_out,
                                      unsigned long long *__restrict__ gmax_bits, unsigned int *__restrict__ bad)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n_xi * n_eta) return;
    const int i = g % n_xi, j = g / n_xi;
    const double hx = 1.0 / (double)(n_xi - 1), hy = 1.0 / (double)(n_eta - 1);
    const int row = j * n_xi, col = i;
    const double u_xi = axis_diff(u, row, i, n_xi, 1, per_xi, 0.0) / hx;
    const double x_xi = axis_diff(x, row, i, n_xi, 1, per_xi, Lx) / hx;
    const double y_xi = axis_diff(y, row, i, n_xi, 1, per_xi, 0.0) / hx;
    const double u_eta = axis_diff(u, col, j, n_eta, n_xi, per_eta, 0.0) / hy;
    const double x_eta = axis_diff(x, col, j, n_eta, n_xi, per_eta, 0.0) / hy;
    const double y_eta = axis_diff(y, col, j, n_eta, n_xi, per_eta, Ly) / hy;
    const double jac = x_xi * y_eta - x_eta * y_xi;
    const double ux = (u_xi * y_eta - u_eta * y_xi) / jac;
    const double uy = (u_eta * x_xi - u_xi * x_eta) / jac;
    const double gg = ux * ux + uy * uy;
    g_out[g] = gg;
    if (!(gg >= 0.0) || gg > 1.0e300) {   // NaN / infinite: vanishing Jacobian or bad input
        atomicOr(bad, 1u);
        return;
    }
    // non-negative doubles order like their bit patterns
    atomicMax(gmax_bits, (unsigned long long)__double_as_longlong(gg));
}

__global__ void arclength_rho_kernel(const double *__restrict__ g_in, int n, double alpha, int normalize,
                                     const unsigned long long *__restrict__ gmax_bits, double *__restrict__ rho)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    double a = alpha;
    if (normalize) {
        const double gmax = __longlong_as_double((long long)*gmax_bits);
        a = gmax > 0.0 ? alpha / gmax : 0.0;
    }
    rho[k] = sqrt(1.0 + a * g_in[k]);
}

// ---------------------------------------------------------------------------
// Mesh quality
// ---------------------------------------------------------------------------
__device__ __forceinline__ double cell_q(const double *x, const double *y, int i, int j, int n_xi, double hx, double hy)
{
    const int g00 = j * n_xi + i, g10 = g00 + 1, g01 = g00 + n_xi, g11 = g01 + 1;
    const double x_xi = 0.5 * ((x[g10] - x[g00]) + (x[g11] - x[g01])) / hx;
    const double y_xi = 0.5 * ((y[g10] - y[g00]) + (y[g11] - y[g01])) / hx;
    const double x_eta = 0.5 * ((x[g01] - x[g00]) + (x[g11] - x[g10])) / hy;
    const double y_eta = 0.5 * ((y[g01] - y[g00]) + (y[g11] - y[g10])) / hy;
    const double tr = x_xi * x_xi + y_xi * y_xi + x_eta * x_eta + y_eta * y_eta;
    const double det = fabs(x_xi * y_eta - x_eta * y_xi);
    return 0.5 * tr / det;
}

// R per cell; per-block maximum and sum (fixed tree order) into partials.
__global__ __launch_bounds__(kQualityBlock) void quality_kernel(const double *__restrict__ xs,
                                                               const double *__restrict__ ys,
                                                               const double *__restrict__ xd,
                                                               const double *__restrict__ yd, int n_xi, int n_eta,
                                                               double *__restrict__ r_cells,
                                                               double *__restrict__ part_max,
                                                               double *__restrict__ part_sum)
{
    __shared__ double smax[kQualityBlock], ssum[kQualityBlock];
    const int nc = (n_xi - 1) * (n_eta - 1);
    const int c = blockIdx.x * kQualityBlock + threadIdx.x;
    double r = 0.0, mx = 0.0;
    if (c < nc) {
        const int i = c % (n_xi - 1), j = c / (n_xi - 1);
        const double hx = 1.0 / (double)(n_xi - 1), hy = 1.0 / (double)(n_eta - 1);
        r = cell_q(xs, ys, i, j, n_xi, hx, hy) / cell_q(xd, yd, i, j, n_xi, hx, hy);
        mx = r;
        if (r_cells) r_cells[c] = r;
    }
    smax[threadIdx.x] = mx;
    ssum[threadIdx.x] = r;
    __syncthreads();
    for (int w = kQualityBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + w]);
            ssum[threadIdx.x] = ssum[threadIdx.x] + ssum[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part_max[blockIdx.x] = smax[0];
        part_sum[blockIdx.x] = ssum[0];
    }
}

// One workgroup: partials in block order -> (max, mean).
__global__ __launch_bounds__(kQualityBlock) void quality_final_kernel(const double *__restrict__ part_max,
                                                                     const double *__restrict__ part_sum,
                                                                     int n_parts, int n_cells,
                                                                     double *__restrict__ out)
{
    __shared__ double smax[kQualityBlock], ssum[kQualityBlock];
    double mx = 0.0, sm = 0.0;
    for (int k = threadIdx.x; k < n_parts; k += kQualityBlock) {
        mx = fmax(mx, part_max[k]);
        sm = sm + part_sum[k];
    }
    smax[threadIdx.x] = mx;
    ssum[threadIdx.x] = sm;
    __syncthreads();
    for (int w = kQualityBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + w]);
            ssum[threadIdx.x] = ssum[threadIdx.x] + ssum[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = smax[0];
        out[1] = ssum[0] / (double)n_cells;
    }
}

inline unsigned blocks_of(size_t n, unsigned b) { return (unsigned)((n + b - 1) / b); }

// ---------------------------------------------------------------------------
// Piecewise-linear transfer of a nodal field between meshes (MᵏP, section 5)
// ---------------------------------------------------------------------------
__device__ __forceinline__ int floor_div(int a, int m) { return a >= 0 ? a / m : -((-a + m - 1) / m); }

// Old-mesh node at grid indices (ii, jj) that may lie beyond a periodic
// seam: wrapped into range, with the period added to the winding coordinate.
__device__ __forceinline__ void old_node(const TransferArgs &a, int ii, int jj, double &x, double &y, double &f)
{
    double ox = 0.0, oy = 0.0;
    if (a.per_xi) {
        const int q = floor_div(ii, a.n_xi - 1);
        ii -= q * (a.n_xi - 1);
        ox = (double)q * a.Lx;
    }
    if (a.per_eta) {
        const int q = floor_div(jj, a.n_eta - 1);
        jj -= q * (a.n_eta - 1);
        oy = (double)q * a.Ly;
    }
    const size_t k = (size_t)jj * a.n_xi + ii;
    x = a.x_old[k] + ox;
    y = a.y_old[k] + oy;
    f = a.f_old[k];
}

// Barycentric test of point p against triangle (A, B, C): the smallest
// coordinate and the linear interpolant of the vertex values.
__device__ __forceinline__ void tri_test(double px, double py, double ax, double ay, double af, double bx, double by,
                                         double bf, double cx, double cy, double cf, double &lmin, double &val)
{
    const double e1x = bx - ax, e1y = by - ay, e2x = cx - ax, e2y = cy - ay;
    const double det = e1x * e2y - e1y * e2x;
    const double dx = px - ax, dy = py - ay;
    const double lb = (dx * e2y - dy * e2x) / det;
    const double lc = (e1x * dy - e1y * dx) / det;
    const double la = 1.0 - lb - lc;
    lmin = fmin(fmin(la, lb), lc);
    val = la * af + lb * bf + lc * cf;
}

// One thread per new node.  The search starts with the 4 x 4 old cells
// around the node's own grid position (a mesh step moves a node by about a
// cell at most) and doubles the window until a triangle contains the point
// (smallest coordinate >= -1e-10: a point on a shared edge or a rounding
// error outside the mesh) or the window covers the whole mesh (with its
// periodic images), so every thread ends.
__global__ void transfer_p1_kernel(TransferArgs a)
{
    const int idx = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (idx >= a.n_xi * a.n_eta) return;
    int i = idx % a.n_xi, j = idx / a.n_xi;
    if (a.per_xi && i == a.n_xi - 1) i = 0;     // image node: node 0's value
    if (a.per_eta && j == a.n_eta - 1) j = 0;
    const double px = a.x_new[(size_t)j * a.n_xi + i], py = a.y_new[(size_t)j * a.n_xi + i];
    const int cxm = a.n_xi - 2, cym = a.n_eta - 2;   // last cell index per axis
    double best = -INFINITY, bval = 0.0;
    for (int w = 2;; w *= 2) {
        int i0 = i - w, i1 = i + w - 1, j0 = j - w, j1 = j + w - 1;
        if (!a.per_xi) {
            i0 = max(i0, 0);
            i1 = min(i1, cxm);
        }
        if (!a.per_eta) {
            j0 = max(j0, 0);
            j1 = min(j1, cym);
        }
        for (int cj = j0; cj <= j1; ++cj) {
            for (int ci = i0; ci <= i1; ++ci) {
                double ax, ay, af, bx, by, bf, cx, cy, cf, dx, dy, df;
                old_node(a, ci, cj, ax, ay, af);
                old_node(a, ci + 1, cj, bx, by, bf);
                old_node(a, ci + 1, cj + 1, cx, cy, cf);
                old_node(a, ci, cj + 1, dx, dy, df);
                double l, v;
                tri_test(px, py, ax, ay, af, bx, by, bf, cx, cy, cf, l, v);
                if (l > best) {
                    best = l;
                    bval = v;
                }
                tri_test(px, py, ax, ay, af, cx, cy, cf, dx, dy, df, l, v);
                if (l > best) {
                    best = l;
                    bval = v;
                }
            }
        }
        if (best >= -1e-10) break;
        const bool all_xi = a.per_xi ? w >= 2 * (a.n_xi - 1) : (i0 == 0 && i1 == cxm);
        const bool all_eta = a.per_eta ? w >= 2 * (a.n_eta - 1) : (j0 == 0 && j1 == cym);
        if (all_xi && all_eta) break;
    }
    a.f_new[idx] = bval;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
size_t edge_gen_lds_bytes(int n_max) { return (size_t)3 * (size_t)n_max * sizeof(double); }

hipError_t launch_edge_gen(const double *rho, const double *rho_xi, const double *rho_eta, int n_xi, int n_eta,
                           int per_xi, int per_eta, double Lx, double Ly, double tau, int L_eta, int L_xi,
                           double *bnd, hipStream_t s)
{
    const int sides = (per_xi ? 0 : 2) + (per_eta ? 0 : 2);
    if (sides == 0) return hipSuccess;
    const int n_max = per_xi ? n_xi : (per_eta ? n_eta : (n_xi > n_eta ? n_xi : n_eta));
    const int block = std::min(kEdgeBlock, (n_max + 63) / 64 * 64);
    const bool p2 = (per_xi || power_of_two(n_eta - 1)) && (per_eta || power_of_two(n_xi - 1));
    if (p2)
        hipLaunchKernelGGL(edge_gen_kernel<true>, dim3(sides), dim3(block), edge_gen_lds_bytes(n_max), s, rho, rho_xi,
                           rho_eta, n_xi, n_eta, per_xi, per_eta, Lx, Ly, tau, L_eta, L_xi, bnd);
    else
        hipLaunchKernelGGL(edge_gen_kernel<false>, dim3(sides), dim3(block), edge_gen_lds_bytes(n_max), s, rho, rho_xi,
                           rho_eta, n_xi, n_eta, per_xi, per_eta, Lx, Ly, tau, L_eta, L_xi, bnd);
    return hipGetLastError();
}

hipError_t launch_targets(const MeshStepArgs &a, double *x_new, double *y_new, hipStream_t s)
{
    const size_t n = (size_t)a.n_xi * a.n_eta;
    hipLaunchKernelGGL(targets_kernel, dim3(blocks_of(n, 256)), dim3(256), 0, s, a, x_new, y_new);
    return hipGetLastError();
}

size_t subdomain_lds_bytes(int P_xi, int P_eta) { return (size_t)2 * (P_xi + 1) * (P_eta + 1) * sizeof(double); }

bool subdomain_fits_lds(int P_xi, int P_eta)
{
    const long nin = (long)(P_xi - 1) * (P_eta - 1);
    const long nb = 2L * (P_xi + 1) + 2L * (P_eta - 1);
    return P_xi >= 2 && P_eta >= 2 && nin <= (long)kSubBlock * kSubPerThread && nb <= kSubBlock &&
           subdomain_lds_bytes(P_xi, P_eta) <= kSubLdsMax;
}

template <bool P2>
static void launch_sub(const MeshStepArgs &a, const SubShape &h, double *x_new, double *y_new, hipStream_t s)
{
    const dim3 grid(a.sub_xi * a.sub_eta), block(h.block);
    const size_t lds = 2 * subdomain_lds_bytes(a.P_xi, a.P_eta);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, s, a, h.inner, h.first_bnd, x_new, y_new); };
    if (h.nodes == 4)
        launch(subdomain_lds_kernel<P2, 4>);
    else if (h.nodes == 3)
        launch(subdomain_lds_kernel<false, 3>);   // (with divisions only)
    else if (h.nodes == 2)
        launch(subdomain_lds_kernel<P2, 2>);
    else
        launch(subdomain_lds_kernel<P2, 1>);
}

hipError_t launch_subdomain_lds(const MeshStepArgs &a, double *x_new, double *y_new, hipStream_t s)
{
    const bool exact = exact_scaling(a.n_xi, a.n_eta);
    const SubShape h = subdomain_shape(a.P_xi, a.P_eta, exact);
    if (!h.block) return hipErrorInvalidValue;
    if (exact)
        launch_sub<true>(a, h, x_new, y_new, s);
    else
        launch_sub<false>(a, h, x_new, y_new, s);
    return hipGetLastError();
}

hipError_t launch_fe_sweep(const MeshStepArgs &a, const double *cx, const double *cy, double *nx, double *ny,
                           double th1, hipStream_t s)
{
    if (a.steps == 0) {
        const size_t n = (size_t)a.n_xi * a.n_eta;
        hipLaunchKernelGGL(fe_sweep_kernel, dim3(blocks_of(n, 256)), dim3(256), 0, s, a, cx, cy, nx, ny, th1);
        return hipGetLastError();
    }
    const bool per = !a.with_interfaces && (a.per_xi || a.per_eta);
    if (a.steps < 1 || a.steps > kTileRim || a.l0 < 0 || a.l0 + a.steps > a.L) return hipErrorInvalidValue;
    const int nix = per && a.per_xi ? a.n_xi - 1 : a.P_xi - 1, niy = per && a.per_eta ? a.n_eta - 1 : a.P_eta - 1;
    const size_t tiles = (size_t)blocks_of((size_t)std::max(nix, 0), kTileCore) *
                         blocks_of((size_t)std::max(niy, 0), kTileCore) * a.sub_xi * a.sub_eta;
    if (tiles == 0) return hipSuccess;   // boxes of one cell: every node is Dirichlet
    if (tiles > 0x7FFFFFFFu) return hipErrorInvalidValue;
    const bool p2 = exact_scaling(a.n_xi, a.n_eta);
    const dim3 grid((unsigned)tiles), block(kTileSide * kTileSide / kTileRows);
    if (p2 && per)
        hipLaunchKernelGGL((fe_tile_kernel<true, true>), grid, block, 0, s, a, cx, cy, nx, ny);
    else if (p2)
        hipLaunchKernelGGL((fe_tile_kernel<true, false>), grid, block, 0, s, a, cx, cy, nx, ny);
    else if (per)
        hipLaunchKernelGGL((fe_tile_kernel<false, true>), grid, block, 0, s, a, cx, cy, nx, ny);
    else
        hipLaunchKernelGGL((fe_tile_kernel<false, false>), grid, block, 0, s, a, cx, cy, nx, ny);
    return hipGetLastError();
}

hipError_t launch_arclength(const double *u, const double *x, const double *y, int n_xi, int n_eta, int per_xi,
                            int per_eta, double Lx, double Ly, double alpha, int normalize, double *g_scratch,
                            unsigned long long *gmax_bits, unsigned int *bad, double *rho, hipStream_t s)
{
    const size_t n = (size_t)n_xi * n_eta;
    hipLaunchKernelGGL(arclength_grad_kernel, dim3(blocks_of(n, 256)), dim3(256), 0, s, u, x, y, n_xi, n_eta, per_xi,
                       per_eta, Lx, Ly, g_scratch, gmax_bits, bad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(arclength_rho_kernel, dim3(blocks_of(n, 256)), dim3(256), 0, s, g_scratch, (int)n, alpha,
                       normalize, gmax_bits, rho);
    return hipGetLastError();
}

hipError_t launch_transfer_p1(const TransferArgs &a, hipStream_t s)
{
    const size_t n = (size_t)a.n_xi * a.n_eta;
    hipLaunchKernelGGL(transfer_p1_kernel, dim3(blocks_of(n, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

int quality_parts(int n_xi, int n_eta) { return (int)blocks_of((size_t)(n_xi - 1) * (n_eta - 1), kQualityBlock); }

hipError_t launch_quality(const double *xs, const double *ys, const double *xd, const double *yd, int n_xi,
                          int n_eta, double *r_cells, double *part_max, double *part_sum, double *out2,
                          hipStream_t s)
{
    const int parts = quality_parts(n_xi, n_eta);
    hipLaunchKernelGGL(quality_kernel, dim3(parts), dim3(kQualityBlock), 0, s, xs, ys, xd, yd, n_xi, n_eta, r_cells,
                       part_max, part_sum);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(quality_final_kernel, dim3(1), dim3(kQualityBlock), 0, s, part_max, part_sum, parts,
                       (n_xi - 1) * (n_eta - 1), out2);
    return hipGetLastError();
}

}  // namespace msdd
