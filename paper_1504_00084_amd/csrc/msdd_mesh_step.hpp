// Device-side interface of the mesh-step kernels (mesh_step.hip): the 1-D
// edge generator, the Dirichlet targets of the decomposed problem, the
// subdomain solves (LDS-resident or global sweeps), the arc-length monitor,
// the mesh-quality ratio and the piecewise-linear monitor transfer of the
// MᵏP variant.  All FP64.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace msdd {

constexpr int kEdgeBlock = 1024;
constexpr int kSubBlock = 1024;                 // one workgroup per subdomain
constexpr int kSubPerThread = 4;                // interior nodes per thread of the LDS solve's size limit
constexpr size_t kSubLdsMax = 160u * 1024u;     // LDS of one CU on gfx950
constexpr int kQualityBlock = 256;
constexpr int kTileCore = 16;                   // the sweeps' tiles: nodes a workgroup advances per axis,
constexpr int kTileRim = 8;                     // the rim around them = substeps per launch,
constexpr int kTileSide = kTileCore + 2 * kTileRim;
constexpr int kTileRows = 2;                    // and nodes per thread

inline bool power_of_two(int n) { return n > 0 && (n & (n - 1)) == 0; }

// Whether both cell counts are powers of two: the updates then need no
// divisions (fe_update).
inline bool exact_scaling(int n_xi, int n_eta) { return power_of_two(n_xi - 1) && power_of_two(n_eta - 1); }

// Workgroup of the LDS solve of one (P_xi + 1) x (P_eta + 1) subdomain that
// subdomain_fits_lds admits: nodes per thread, the threads that own interior
// nodes, the first one that owns a boundary node, the block, and the node
// updates that follow one another on a SIMD.  Where the workgroup has too few
// threads for both, its last threads own interior and boundary nodes.
// block = 0 for other subdomains.
// Without divisions (`exact`) a thread owns a segment of a column, which saves
// LDS reads: as many rows as leave the fewest updates in a row, of equal ones
// two, then one (33 x 33 boxes, 300 substeps: two rows 151 us, one 169, four
// 181).  With divisions the updates bound the solve, so the nodes are dealt
// out evenly, one to four to a thread: 48 x 48 cells 9 updates in a row, 12
// in segments of four.  41 x 41 boxes, 300 substeps: 557 us, in segments of
// four 699, of eight, which spilled registers, 756.
struct SubShape {
    int nodes, inner, first_bnd, block, cost;
};
inline SubShape subdomain_shape(int P_xi, int P_eta, bool exact)
{
    const long nin = (long)(P_xi - 1) * (P_eta - 1), nb = 2L * (P_xi + 1) + 2L * (P_eta - 1), bnd = (nb + 63) / 64 * 64;
    SubShape best{0, 0, 0, 0, 0};
    if (P_xi < 2 || P_eta < 2 || nb > kSubBlock || nin > (long)kSubBlock * kSubPerThread ||
        (size_t)4 * (P_xi + 1) * (P_eta + 1) * sizeof(double) > kSubLdsMax)
        return best;
    auto take = [&](int nodes, long threads, long cost) {
        const long inner = (threads + 63) / 64 * 64, first = inner + bnd > kSubBlock ? kSubBlock - bnd : inner;
        if (inner > kSubBlock || (best.block && cost >= best.cost)) return;
        best = SubShape{nodes, (int)inner, (int)first, (int)(first + bnd > inner ? first + bnd : inner), (int)cost};
    };
    if (exact) {
        for (int rows : {2, 1, 4}) {
            if (P_eta - 1 < rows) continue;
            const long segs = (long)(P_xi - 1) * ((P_eta - 1 + rows - 1) / rows);
            take(rows, segs, (segs + 255) / 256 * rows);
        }
    } else {
        const long full = (nin - 1) / kSubBlock;   // nodes that every thread owns
        take((int)full + 1, full ? kSubBlock : nin, 4 * full + (nin - full * kSubBlock + 255) / 256);
    }
    return best;
}

// Whether tiles of the whole grid advance subdomains faster than one
// workgroup for each does, by the time of a substep on `cus` compute units:
// a workgroup's updates one after the other (80 ns each without divisions,
// 270 with them; 220 ns for threads that own boundary nodes as well), or an
// eighth of a launch (630 ns) and the tiles that follow one another on a
// compute unit.  4 x 4 boxes of 61 x 61, 300 substeps: LDS 1210 us, tiles 580;
// 2 x 2 of 65 x 65 without divisions 429 and 326; 12 x 12 of 42 x 42, 100
// substeps: LDS 225 us, tiles 781.
inline bool subdomain_tiles(int P_xi, int P_eta, long boxes, long cus, const SubShape &h, bool exact)
{
    const long tiles = boxes * ((P_xi - 1 + kTileCore - 1) / kTileCore) * ((P_eta - 1 + kTileCore - 1) / kTileCore);
    const long lds = (boxes + cus - 1) / cus *
                     ((exact ? 100 + 80 * (long)h.cost : 30 + 270 * (long)h.cost) + (h.first_bnd < h.inner ? 220 : 0));
    return lds > 630 + (tiles + cus - 1) / cus * (exact ? 420 : 1160);
}

// Everything the targets / subdomain / sweep kernels read; device pointers.
struct MeshStepArgs {
    int n_xi, n_eta, sub_xi, sub_eta, P_xi, P_eta;
    int per_xi, per_eta, with_interfaces, L;
    double Lx, Ly, tau;
    const double *x0, *y0;                 // mesh at t^n [n_eta][n_xi]
    const double *bnd1;                    // boundary arrays at t^{n+1}
    const double *iface_x, *iface_y;       // interface estimate at t^{n+1}, by rank
    const int32_t *node_rank;              // [n_eta][n_xi]: interface rank or -1
    const double *rho, *rho_xi, *rho_eta;  // FP64 node tables of the frozen monitor
    double *tx1, *ty1;                     // Dirichlet values at t^{n+1}, the drift coefficients rho_xi / rho and
                                           // rho_eta / rho of the other nodes (written by the targets kernel)
    uint8_t *mask;                         // 1 on Dirichlet nodes
    int l0, steps;                         // launch_fe_sweep: substeps done, substeps of this launch (0: the
                                           // plain sweep of one substep)
};

size_t edge_gen_lds_bytes(int n_max);
hipError_t launch_edge_gen(const double *rho, const double *rho_xi, const double *rho_eta, int n_xi, int n_eta,
                           int per_xi, int per_eta, double Lx, double Ly, double tau, int L_eta, int L_xi,
                           double *bnd, hipStream_t s);
hipError_t launch_targets(const MeshStepArgs &a, double *x_new, double *y_new, hipStream_t s);
size_t subdomain_lds_bytes(int P_xi, int P_eta);
bool subdomain_fits_lds(int P_xi, int P_eta);
hipError_t launch_subdomain_lds(const MeshStepArgs &a, double *x_new, double *y_new, hipStream_t s);
hipError_t launch_fe_sweep(const MeshStepArgs &a, const double *cx, const double *cy, double *nx, double *ny,
                           double th1, hipStream_t s);
hipError_t launch_arclength(const double *u, const double *x, const double *y, int n_xi, int n_eta, int per_xi,
                            int per_eta, double Lx, double Ly, double alpha, int normalize, double *g_scratch,
                            unsigned long long *gmax_bits, unsigned int *bad, double *rho, hipStream_t s);
// MᵏP monitor update (section 5): f at the nodes of a new mesh from the
// piecewise-linear interpolant of nodal values on an old mesh of the same
// grid.  Each old cell (i, j)-(i+1, j+1) is split along its diagonal from
// node (i, j) to node (i+1, j+1); a point takes the linear interpolant of
// the triangle that contains it (outside the old mesh: of the triangle
// whose smallest barycentric coordinate is largest).  Periodic axes extend
// the old mesh by its images (+Lx along xi, +Ly along eta); image nodes of
// the new mesh take node 0's value.
struct TransferArgs {
    int n_xi, n_eta, per_xi, per_eta;
    double Lx, Ly;
    const double *x_old, *y_old, *f_old;   // [n_eta][n_xi]
    const double *x_new, *y_new;
    double *f_new;
};
hipError_t launch_transfer_p1(const TransferArgs &a, hipStream_t s);

int quality_parts(int n_xi, int n_eta);
hipError_t launch_quality(const double *xs, const double *ys, const double *xd, const double *yd, int n_xi,
                          int n_eta, double *r_cells, double *part_max, double *part_sum, double *out2,
                          hipStream_t s);

}  // namespace msdd
