// FP64 path arithmetic and the wave loop of the FP64 path kernel (device
// code, included by kernels.hip): the estimator of section 3.4 with every
// quantity in double precision.
#pragma once

namespace msdd {

// ---------------------------------------------------------------------------
// Elementary functions on the argument sets a path needs
// ---------------------------------------------------------------------------
// The two normals of a substep come from 23-bit uniforms, so their functions
// take the 24-bit odd integer of the uniform and skip every special case of
// the library's: no subnormals, no infinities, no range reduction beyond an
// exact one.  The polynomials interpolate the function at Chebyshev nodes in
// 60-digit arithmetic; the errors stated are against 60-digit values, before
// the rounding of the evaluation.

// A constant in scalar registers, set where it is used: two scalar moves, which
// issue beside the vector instructions of the SIMD's other waves.  Left alone
// the compiler keeps the two dozen polynomial coefficients in 36 vector
// registers across the loop and copies each into place ahead of its
// multiply-add (20 more vector instructions per substep, and spills).
__device__ __forceinline__ double sconst(double c)
{
    asm volatile("" : "+s"(c));
    return c;
}

// 1 / b to the last bits: the hardware reciprocal (better than 2^-20) and two
// Newton steps.  b positive and far from the ends of the exponent range.
__device__ __forceinline__ double rcp64(double b)
{
    double y = __builtin_amdgcn_rcp(b);
    y = fma(y, fma(-b, y, 1.0), y);
    return fma(y, fma(-b, y, 1.0), y);
}

// sqrt(a), a positive and far from the ends of the exponent range: the
// hardware reciprocal square root, one coupled Newton step for sqrt(a) and
// 1 / (2 sqrt(a)), and a last correction from the exact residual.
__device__ __forceinline__ double sqrt64(double a)
{
    const double y = __builtin_amdgcn_rsq(a);
    double g = a * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, a), h, g);
}

// log(u), u = (2 floor(w / 2^9) + 1) 2^-24.  The odd integer is exact in
// FP32, whose bits give u = 2^e f with f in [sqrt(1/2), sqrt(2)) (the split of
// FreeBSD's and musl's logf: add the bits of 1, take off those of sqrt(1/2)); f - 1 and
// f + 1 are exact, s = (f - 1) / (f + 1), log f = 2 s + s^3 P(s^2) (the atanh
// series; P of degree 6, error below 4e-16 of a term that is at most 1e-2 of
// the result).
__device__ __forceinline__ double log_u(uint32_t w)
{
    uint32_t ix = __float_as_uint((float)((w >> 8) | 1u));
    ix += 0x3F800000u - 0x3F3504F3u;
    const int e = (int)(ix >> 23) - (127 + 24);
    const float f = __uint_as_float((ix & 0x7FFFFFu) + 0x3F3504F3u);
    const double a = (double)(f - 1.0f), b = a + 2.0;
    double y = __builtin_amdgcn_rcp(b);
    y = fma(y, fma(-b, y, 1.0), y);
    double s = a * y;
    s = fma(fma(-b, s, a), y, s);   // the quotient, corrected by its exact residual
    const double z = s * s;
    double p = fma(z, sconst(0x1.2b5900de53b32p-3), 0x1.39fe51a7c18f9p-3);
    p = fma(p, z, sconst(0x1.7462b51cb66b1p-3));
    p = fma(p, z, sconst(0x1.c71c62e3f11e6p-3));
    p = fma(p, z, sconst(0x1.2492492df281ap-2));
    p = fma(p, z, sconst(0x1.99999999952d7p-2));
    p = fma(p, z, sconst(0x1.5555555555558p-1));
    return fma((double)e, sconst(0x1.62e42fefa39efp-1), fma(s * z, p, s + s));
}

// cos and sin of 2 pi u, u = (2 floor(w / 2^9) + 1) 2^-24: the nearest
// quarter turn is split off the integer exactly, the rest r lies in
// [-1/2, 1/2] quarter turns (sin: r times a degree-6, cos: a degree-7
// polynomial in r^2, errors below 1e-16; r is kept as an integer, its scale
// 2^-22 folded into the coefficients, which stay exact).
__device__ __forceinline__ void cos_sin_u(uint32_t w, double &cs, double &sn)
{
    const uint32_t m = (w >> 8) | 1u;
    const uint32_t q = (m + (1u << 21)) >> 22;                // quarter turns, 0..4
    const double r = (double)((int)m - (int)(q << 22));       // 2^22 r
    const double z = r * r;
    double s = fma(z, sconst(0x1.e3f38399551bfp-25 * 0x1p-286), -0x1.e30071afc3e59p-19 * 0x1p-242);
    s = fma(s, z, sconst(0x1.50782fda12d96p-13 * 0x1p-198));
    s = fma(s, z, sconst(-0x1.32d2cce2e5b19p-8 * 0x1p-154));
    s = fma(s, z, sconst(0x1.466bc677587f8p-4 * 0x1p-110));
    s = fma(s, z, sconst(-0x1.4abbce625be41p-1 * 0x1p-66));
    s = fma(s, z, sconst(0x1.921fb54442d18p+0 * 0x1p-22));
    s = s * r;
    double c = fma(z, sconst(-0x1.b2f3eb054afcdp-28 * 0x1p-308), 0x1.f9ce245cada0bp-22 * 0x1p-264);
    c = fma(c, z, sconst(-0x1.a6d1eef479be1p-16 * 0x1p-220));
    c = fma(c, z, sconst(0x1.e1f5068688d5bp-11 * 0x1p-176));
    c = fma(c, z, sconst(-0x1.55d3c7e3cb241p-6 * 0x1p-132));
    c = fma(c, z, sconst(0x1.03c1f081b5ac0p-2 * 0x1p-88));
    c = fma(c, z, sconst(-0x1.3bd3cc9be45dep+0 * 0x1p-44));
    c = fma(c, z, 1.0);
    const bool odd = q & 1u;
    const double a = odd ? s : c, b = odd ? c : s;
    // signs by quarter: cos + - - +, sin + + - -
    const uint32_t fc = ((q + 1u) & 2u) << 30, fs = (q & 2u) << 30;
    cs = __hiloint2double((int)((uint32_t)__double2hiint(a) ^ fc), __double2loint(a));
    sn = __hiloint2double((int)((uint32_t)__double2hiint(b) ^ fs), __double2loint(b));
}

// exp(-a), a >= 0 (1e-304 from 700 on): a = -(k ln 2 + r), |r| <= ln(2) / 2,
// exp(r) = 1 + r + r^2 Q(r) with Q of degree 10 (error below 3e-18).
__device__ __forceinline__ double exp_neg(double a)
{
    a = fmin(a, 700.0);
    const double k = rint(a * sconst(-0x1.71547652b82fep+0));
    double r = fma(-k, sconst(0x1.62e42fefa39efp-1), -a);
    r = fma(-k, sconst(0x1.abc9e3b39803fp-56), r);
    double p = fma(r, sconst(0x1.1f7301a8efa5cp-29), 0x1.af4de6a36d4fcp-26);
    p = fma(p, r, sconst(0x1.27e4db653346ep-22));
    p = fma(p, r, sconst(0x1.71de0232f4775p-19));
    p = fma(p, r, sconst(0x1.a01a01a6d84aap-16));
    p = fma(p, r, sconst(0x1.a01a01abe78f9p-13));
    p = fma(p, r, sconst(0x1.6c16c16c162d5p-10));
    p = fma(p, r, sconst(0x1.11111111100dcp-7));
    p = fma(p, r, sconst(0x1.5555555555556p-5));
    p = fma(p, r, sconst(0x1.5555555555557p-3));
    p = fma(p, r, 0.5);
    return ldexp(fma(r * r, p, r) + 1.0, (int)k);
}

// ---------------------------------------------------------------------------
// Constants, path state, monitor table
// ---------------------------------------------------------------------------
// (The doubles stay in vector registers: forced into scalar ones, of which the
// Philox round keys take 20, the compiler fetched each back from a vector lane
// at every use, 17 instructions more per substep: 129^2 bump 21.9 -> 20.8 ms.)
struct ConstD {
    int nx1, ny1, K, per_xi, per_eta, bridge;
    double fnx1, fny1, lx, ly;    // cells per axis; the largest double below each
    double dt, inv_dt, four_dt;   // -four_dt log u = (sqrt(2 dt) sqrt(-2 log u))^2
    double gx, gy;                // dt / (2 h) per axis: scales the nodal differences of rho
    double delta;                 // farther from every Dirichlet side, no bridge crossing can matter
    const GLOBAL double *pad;     // padded rho, node (0, 0), row stride n_xi + 2
    int stride;
};

// PER >= 0: the periodic flags as compile-time constants (PER & 1: xi,
// PER >> 1: eta); PER < 0: from I.
template <int PER>
__device__ __forceinline__ ConstD load_const_d(const InstView &I)
{
    ConstD c;
    c.nx1 = I.n_xi - 1;
    c.ny1 = I.n_eta - 1;
    c.K = I.K;
    c.per_xi = PER < 0 ? I.per_xi : (PER & 1);
    c.per_eta = PER < 0 ? I.per_eta : (PER >> 1);
    c.bridge = I.bridge;
    c.fnx1 = (double)c.nx1;
    c.fny1 = (double)c.ny1;
    c.lx = c.fnx1 - c.fnx1 * 0x1p-53;
    c.ly = c.fny1 - c.fny1 * 0x1p-53;
    c.dt = I.dt;
    c.inv_dt = 1.0 / I.dt;
    c.four_dt = 4.0 * I.dt;
    c.gx = 0.5 * I.dt * c.fnx1;
    c.gy = 0.5 * I.dt * c.fny1;
    c.delta = sqrt(18.5 * I.dt);
    c.stride = I.n_xi + 2;
    c.pad = gptr(I.rho_pad) + (uint32_t)(c.stride + 1);
    return c;
}

struct PathD {
    double x, y;     // position (periodic axes wrapped)
    double wx, wy;   // winding numbers
    int k;           // substeps done
    bool near;       // nearer than delta to a Dirichlet side
};

// Where the monitor is read.  The drift of a substep takes rho and the
// centred differences of rho at the four corners of a cell: twelve values of
// the padded rho table (rows cy - 1 .. cy + 2 of the cell's two inner and two
// outer columns).  The ghost rows hold 3 f0 - 3 f1 + f2, for which the centred
// difference is the one-sided second-order difference at a Dirichlet side
// ((-3 f0 + 4 f1 - f2) / 2h), and the images on a periodic axis, so one form
// serves every cell and neither gradient table is read: 8 bytes per node in
// LDS instead of 24, which holds a whole grid up to 141 x 141 nodes.
//   mode 0: global memory; mode 1: the whole table in LDS; mode 2: a window
//   of it in LDS, lanes outside the window read global memory.
struct Tab64 {
    const double *lds;   // node (i0, j0) of the window
    int stride;          // of the window's rows
    int i0, j0, w1, h1;  // origin and cells of the window
};

template <class P>
__device__ __forceinline__ void corners64(P p, int s, double *v)
{
    v[0] = p[-1], v[1] = p[0], v[2] = p[1], v[3] = p[2];                       // row cy
    v[4] = p[s - 1], v[5] = p[s], v[6] = p[s + 1], v[7] = p[s + 2];            // row cy + 1
    v[8] = p[-s], v[9] = p[1 - s];                                             // row cy - 1
    v[10] = p[2 * s], v[11] = p[2 * s + 1];                                    // row cy + 2
}

__device__ __forceinline__ double lerp64(double t, double a, double b) { return fma(t, b - a, a); }

__device__ __forceinline__ double side_distance64(const ConstD &C, double x, double y)
{
    const double mx = C.per_xi ? 1.0e300 : fmin(x, 1.0 - x);
    const double my = C.per_eta ? 1.0e300 : fmin(y, 1.0 - y);
    return C.per_xi ? my : (C.per_eta ? mx : fmin(mx, my));
}

__device__ __forceinline__ void wrap64(double &x, double &w)
{
    double f = floor(x);
    x -= f;
    if (x >= 1.0) {   // a tiny negative coordinate plus one
        x -= 1.0;
        f += 1.0;
    }
    w += f;
}

// One EM substep (a3-a6); returns the exit side or -1.  An exited path keeps
// the end of the substep as its position (value64 moves it onto the side).
template <int MODE>
__device__ __forceinline__ int substep64(PathD &P, const ConstD &C, const Tab64 &T, uint32_t wa, uint32_t wb,
                                         uint32_t wc, double *trace4)
{
    double cs, sn;
    cos_sin_u(wb, cs, sn);
    const double rad = sqrt64(-C.four_dt * log_u(wa));

    // Cell and local coordinate.  A coordinate below 1 times the cell count
    // stays below the count; exactly 1, on a Dirichlet side, takes the last
    // cell at the largest local coordinate below 1.
    const double sx = C.per_xi ? P.x * C.fnx1 : fmin(P.x * C.fnx1, C.lx);
    const double sy = C.per_eta ? P.y * C.fny1 : fmin(P.y * C.fny1, C.ly);
    const int cx = (int)sx, cy = (int)sy;
    const double tx = __builtin_amdgcn_fract(sx), ty = __builtin_amdgcn_fract(sy);
    double v[12];
    if (MODE == 0) {
        corners64(C.pad + (int64_t)cy * C.stride + cx, C.stride, v);
    } else if (MODE == 1) {
        corners64(T.lds + (int)__umul24((uint32_t)cy, (uint32_t)T.stride) + cx, T.stride, v);
    } else {
        const int rx = cx - T.i0, ry = cy - T.j0;
        if (((uint32_t)rx >= (uint32_t)T.w1) | ((uint32_t)ry >= (uint32_t)T.h1))
            corners64(C.pad + (int64_t)cy * C.stride + cx, C.stride, v);
        else
            corners64(T.lds + (int)__umul24((uint32_t)ry, (uint32_t)T.stride) + rx, T.stride, v);
    }
    const double rho = lerp64(ty, lerp64(tx, v[1], v[2]), lerp64(tx, v[5], v[6]));
    const double dx = lerp64(ty, lerp64(tx, v[2] - v[0], v[3] - v[1]), lerp64(tx, v[6] - v[4], v[7] - v[5]));
    const double dy = lerp64(ty, lerp64(tx, v[5] - v[8], v[6] - v[9]), lerp64(tx, v[10] - v[1], v[11] - v[2]));
    const double inv = rcp64(rho);
    double nx = fma(rad, cs, fma(dx * inv, C.gx, P.x));
    double ny = fma(rad, sn, fma(dy * inv, C.gy, P.y));

    if (C.per_xi) wrap64(nx, P.wx);
    if (C.per_eta) wrap64(ny, P.wy);
    if (trace4) {
        const double sq = sqrt(2.0 * C.dt);
        trace4[0] = nx;
        trace4[1] = ny;
        trace4[2] = rad * cs / sq;
        trace4[3] = rad * sn / sq;
    }
    const double m = side_distance64(C, nx, ny);
    const bool near = m < C.delta;
    int side = -1;
    if (m < 0.0) {
        side = !C.per_xi && nx < 0.0 ? 0 : (!C.per_xi && nx > 1.0 ? 1 : (!C.per_eta && ny < 0.0 ? 2 : 3));
    } else if (C.bridge && (near || P.near)) {
        // Both ends farther than delta from a side: its crossing probability
        // is below exp(-18.5) = 9.2e-9, and four such sides together below the
        // smallest uniform (6e-8), so the test cannot succeed.
        const double big = 1.0e300;
        const double a0 = C.per_xi ? big : P.x * nx * C.inv_dt, a1 = C.per_xi ? big : (1.0 - P.x) * (1.0 - nx) * C.inv_dt;
        const double a2 = C.per_eta ? big : P.y * ny * C.inv_dt, a3 = C.per_eta ? big : (1.0 - P.y) * (1.0 - ny) * C.inv_dt;
        const double ax = a1 < a0 ? a1 : a0, ay = a3 < a2 ? a3 : a2;
        if (ax < 18.5 || ay < 18.5) {
            // a side beyond 40 has 1 - p = 1 exactly, so the far side of each
            // axis is evaluated only when it is nearer than that (substeps
            // above a few 1e-3, or a drift that crosses the domain)
            const double px = exp_neg(ax), py = exp_neg(ay);
            double stay = (1.0 - px) * (1.0 - py);
            const double fx = a1 < a0 ? a0 : a1, fy = a3 < a2 ? a2 : a3;
            if (fx < 40.0 || fy < 40.0) stay *= (1.0 - exp_neg(fx)) * (1.0 - exp_neg(fy));
            if (uniform_f64(wc) < 1.0 - stay) side = py > px ? (a3 < a2 ? 3 : 2) : (a1 < a0 ? 1 : 0);
        }
    }
    P.x = nx;
    P.y = ny;
    P.near = near;
    return side;
}

// Value of an ended path (a7), winding offsets included.
__device__ __forceinline__ void value64(const InstView &I, const ConstD &C, const PathD &P, int side, double &vx,
                                        double &vy)
{
    if (side >= 0) {
        const double w_tn = (double)P.k * C.dt / I.tau;
        const double tang = fmin(fmax(side < 2 ? P.y : P.x, 0.0), 1.0);
        vx = boundary_d(I.bnd0, I.bnd1, I.n_xi, I.n_eta, side, 0, tang, w_tn);
        vy = boundary_d(I.bnd0, I.bnd1, I.n_xi, I.n_eta, side, 1, tang, w_tn);
    } else {
        vx = keys_d(I.xpad, I.n_xi, I.n_eta, P.x, P.y);
        vy = keys_d(I.ypad, I.n_xi, I.n_eta, P.x, P.y);
    }
    if (C.per_xi) vx += P.wx * I.Lx;
    if (C.per_eta) vy += P.wy * I.Ly;
}

// Advances one path by groups of four substeps (three Philox blocks), up to
// `quarters` of them, until fewer than `lanes` of the wave's lanes still
// have a path in flight.  Sets `ended` when the path left or reached K.
template <bool TRACE, int MODE>
__device__ __forceinline__ int group64(PathD &P, const ConstD &C, const Tab64 &T, uint32_t path, uint32_t node,
                                       uint32_t ctr3, uint32_t key0, uint32_t key1, bool &ended, double *trace,
                                       uint32_t quarters, uint32_t lanes)
{
    int side = -1;
    ended = false;
#pragma unroll 1
    for (uint32_t q = 0; q < quarters; ++q) {
        if (q > 0 && (uint32_t)__popcll(__ballot(!ended && P.k < C.K)) < lanes) break;
        const uint32_t blk = 3u * ((uint32_t)P.k >> 2);
        const Words4 A = philox4x32_10(blk, path, node, ctr3, key0, key1);
        const Words4 B = philox4x32_10(blk + 1u, path, node, ctr3, key0, key1);
        const Words4 G = philox4x32_10(blk + 2u, path, node, ctr3, key0, key1);
        const uint32_t w[12] = {A.w0, A.w1, A.w2, A.w3, B.w0, B.w1, B.w2, B.w3, G.w0, G.w1, G.w2, G.w3};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (!ended && P.k < C.K) {
                double t4[4];
                side = substep64<MODE>(P, C, T, w[3 * s], w[3 * s + 1], w[3 * s + 2], TRACE ? t4 : nullptr);
                if (TRACE) {
                    double *t = trace + 4 * (size_t)P.k;
                    t[0] = t4[0];
                    t[1] = t4[1];
                    t[2] = t4[2];
                    t[3] = t4[3];
                }
                P.k += 1;
                ended = side >= 0;
            }
        }
    }
    ended = ended || P.k >= C.K;
    return side;
}

// ---------------------------------------------------------------------------
// Wave loop
// ---------------------------------------------------------------------------
// Lane l of the wave runs paths l, l + 64, ... of each of the wave's items, in
// that order, and goes on to the next item as soon as its share of the
// current one is done: lanes whose paths leave early do not wait for the
// wave, as long as they are at most one item ahead.  A lane's sums are those
// of its own paths in their order, so an item's totals depend neither on
// the schedule nor on which wave ran it, and no path needs its end state
// stored.  Two items are in flight per wave; the older one is reduced and
// written once every lane has left it.  Over all vector instructions 78 % of
// the lanes take part on the 129^2 bump (15 % of whose path-steps are saved by
// exits).  The stepping loop
// is left once fewer than 48 lanes are busy (56 and 60: 1 and 2 % slower).
struct Item64 {
    uint32_t node, p_begin, count, partial;
};

template <int PER, int MODE, class Src>
__device__ __forceinline__ void item_loop64(Src &src, const InstView &I, const ConstD &C, const Tab64 &T, int lane)
{
    const uint32_t key0 = I.key0, key1 = I.key1, ctr3 = I.ctr3;
    GLOBAL Partial *const partials = gptr_rw(I.partials);
    Item64 it0{0u, 0u, 0u, 0u}, it1{0u, 0u, 0u, 0u};   // items of even and odd number
    uint32_t head = 0, loaded = 0;   // oldest item in flight, items taken so far
    bool more = true;
    // lane state (the node's position and mesh values are read again where a
    // path starts or ends: registers are what limits this kernel)
    bool has = false;
    uint32_t ls = 0, t = (uint32_t)lane, path = 0, rank = 0;   // own item number, next path in it
    PathD P{0.0, 0.0, 0.0, 0.0, 0, false};
    double c1x = 0.0, c2x = 0.0, c1y = 0.0, c2y = 0.0, o1x = 0.0, o2x = 0.0, o1y = 0.0, o2y = 0.0;
    uint32_t cex = 0, oex = 0;
    unsigned long long cst = 0, ost = 0;

    for (;;) {
        // take items until two are in flight
        while (more && loaded - head < 2u) {
            Item64 it;
            more = src.next(lane, it.node, it.p_begin, it.count, it.partial);
            if (!more) break;
            if (loaded & 1u)
                it1 = it;
            else
                it0 = it;
            ++loaded;
        }
        // lanes without a path: on to the next item when theirs has none left
        // for them, then the next path of their item
        if (!has) {
            if (ls == head && ls < loaded && t >= ((ls & 1u) ? it1.count : it0.count)) {
                o1x = c1x, o2x = c2x, o1y = c1y, o2y = c2y, oex = cex, ost = cst;
                c1x = c2x = c1y = c2y = 0.0;
                cex = 0;
                cst = 0;
                ++ls;
                t = (uint32_t)lane;
            }
            const bool odd = ls & 1u;
            if (ls < loaded && t < (odd ? it1.count : it0.count)) {
                has = true;
                path = (odd ? it1.p_begin : it0.p_begin) + t;
                t += 64u;
                const uint32_t node = odd ? it1.node : it0.node;
                rank = gptr(I.node_r)[node];
                P.x = (double)gptr(I.node_i)[node] / C.fnx1;
                P.y = (double)gptr(I.node_j)[node] / C.fny1;
                P.near = side_distance64(C, P.x, P.y) < C.delta;
                P.wx = 0.0;
                P.wy = 0.0;
                P.k = 0;
            }
        }
        // every lane has left the oldest item: reduce it
        if (head < loaded && __ballot(ls == head) == 0) {
            const double a = wave_sum(o1x), b = wave_sum(o2x), c = wave_sum(o1y), d = wave_sum(o2y);
            const unsigned long long ex = wave_sum_u64((unsigned long long)oex), st = wave_sum_u64(ost);
            GLOBAL Partial *out = partials + ((head & 1u) ? it1.partial : it0.partial);
            if (lane == 0) {
                out->s1x = a;
                out->s2x = b;
                out->s1y = c;
                out->s2y = d;
                out->exits = ex;
                out->steps = st;
            }
            ++head;
            continue;
        }
        if (__ballot(has) == 0) {
            if (head == loaded && !more) break;
            continue;
        }
        bool ended = false;
        if (has) {
            const int side = group64<false, MODE>(P, C, T, path, rank, ctr3, key0, key1, ended, nullptr, 16u, 48u);
            if (ended) {
                double vx, vy;
                value64(I, C, P, side, vx, vy);
                const uint32_t node = (ls & 1u) ? it1.node : it0.node;
                const size_t g = (size_t)gptr(I.node_j)[node] * (I.n_xi + 2) + gptr(I.node_i)[node];
                const double dx = vx - gptr(I.x64)[g], dy = vy - gptr(I.y64)[g];
                c1x += dx;
                c2x = fma(dx, dx, c2x);
                c1y += dy;
                c2y = fma(dy, dy, c2y);
                cex += side >= 0 ? 1u : 0u;
                cst += (unsigned long long)P.k;
                has = false;
            }
        }
    }
}

}  // namespace msdd
