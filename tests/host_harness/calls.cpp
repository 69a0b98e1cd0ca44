// Host-only checks of what the library's calls hand to its kernels and of
// what they charge to the memory budget (built with g++ against the CPU
// stand-in HIP header; no GPU).  The stub launchers of stub_kernels.cpp, some
// of them recording their arguments.  TEST INFRASTRUCTURE ONLY.  Scenarios
// (argv[1]):
//   arrays   device arrays that kernels may not address are staged
//   budget   requests in slices of 64 paths claim memory only where the budget
//            has room for it beside everything else
//   boxes    a forced LDS solve runs the LDS kernel for every subdomain that
//            fits it, with threads for all its nodes
//   jobs     the jobs of windowed launches hold every item once; those of a
//            launch with few items are as many as its workgroups, or two or
//            three times that, and of one size
//   slices   no slices of 64 paths where many of their lanes would have no path
//   fp64     FP64 requests are charged for the partial sums that they allocate
// Exit status 0 when every check holds; a message names the first failure.
#define launch_prep_mesh stub_launch_prep_mesh
#define launch_finalize stub_launch_finalize
#define launch_subdomain_lds stub_launch_subdomain_lds
#define launch_fe_sweep stub_launch_fe_sweep
#define launch_paths_fp32_window stub_launch_paths_fp32_window
#include "stub_kernels.cpp"
#undef launch_subdomain_lds
#undef launch_fe_sweep
#undef launch_paths_fp32_window
#undef launch_prep_mesh
#undef launch_finalize

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <string>
#include <utility>
#include <vector>

#include "mesh_sdd.h"

static int g_failures = 0;
static void check(bool ok, const char *fmt, ...)
{
    if (ok) return;
    va_list ap;
    va_start(ap, fmt);
    std::vfprintf(stderr, fmt, ap);
    va_end(ap);
    std::fprintf(stderr, " (last error: %s)\n", mesh_sdd_last_error());
    ++g_failures;
}

// ---- recording launchers ---------------------------------------------------
static const double *g_prep_x = nullptr;         // mesh that the last launch_prep_mesh read
static double g_prep_first = 0.0;                // and its first value
static std::vector<const double *> g_final;      // result arrays of the last launch_finalize
static std::vector<uint32_t> g_slices;           // slices per chunk of each request finalized
static uint32_t g_items = 0;                     // items per node of the last one
static mesh_sdd_ctx *g_watched = nullptr;        // its memory in use at every staging, the most
static std::atomic<uint64_t> g_most_in_use{0}, g_most_running{0};
static std::vector<msdd::WinJob> g_jobs;         // of the last windowed launch, with its queues and ranges
static msdd::JobQueues g_queues;
static std::vector<msdd::WorkRange> g_ranges;
static int g_lds_solves = 0, g_sweeps = 0;       // launches of the subdomain solves
static std::mutex g_gate;                        // held: staging waits

namespace msdd {
hipError_t launch_prep_mesh(const double *x, const double *y, int n_xi, int n_eta, int per_xi, int per_eta, double Lx,
                            double Ly, double *xpad, double *ypad, float *xpad_f, float *ypad_f, hipStream_t s)
{
    g_prep_x = x;
    g_prep_first = x[0];
    if (g_watched) {
        std::lock_guard<std::mutex> hold(g_gate);
        mesh_sdd_stats st;
        std::memset(&st, 0, sizeof st);
        st.struct_size = sizeof st;
        mesh_sdd_ctx_stats(g_watched, &st);
        g_most_in_use = std::max<uint64_t>(g_most_in_use, st.hbm_in_use);
        g_most_running = std::max<uint64_t>(g_most_running, st.running);
    }
    return stub_launch_prep_mesh(x, y, n_xi, n_eta, per_xi, per_eta, Lx, Ly, xpad, ypad, xpad_f, ypad_f, s);
}
hipError_t launch_finalize(const Partial *p, const NodeSpan *sp, const InstView *v, uint32_t M, uint64_t n, double *mx,
                           double *my, double *sx, double *sy, double *ef, unsigned long long *t, hipStream_t s)
{
    g_final = {mx, my, sx, sy, ef};
    g_slices.push_back(v->slices);
    g_items = sp->count;
    return stub_launch_finalize(p, sp, v, M, n, mx, my, sx, sy, ef, t, s);
}
hipError_t launch_paths_fp32_window(const InstView *v, const WorkRange *r, const WinJob *j, const JobQueues &qs,
                                    uint32_t *head, uint32_t cap, int kind, size_t lds, int grid, float *ends,
                                    uint32_t waves, uint32_t lanes, uint32_t quarters, hipStream_t s)
{
    g_jobs.assign(j, j + qs.b[kJobQueues]);
    g_queues = qs;
    uint32_t n = 0;
    for (const WinJob &job : g_jobs) n = std::max(n, job.range + 1);
    g_ranges.assign(r, r + n);
    return stub_launch_paths_fp32_window(v, r, j, qs, head, cap, kind, lds, grid, ends, waves, lanes, quarters, s);
}
hipError_t launch_subdomain_lds(const MeshStepArgs &a, double *x, double *y, hipStream_t s)
{
    ++g_lds_solves;
    return stub_launch_subdomain_lds(a, x, y, s);
}
hipError_t launch_fe_sweep(const MeshStepArgs &a, const double *cx, const double *cy, double *nx, double *ny,
                           double th1, hipStream_t s)
{
    ++g_sweeps;
    return stub_launch_fe_sweep(a, cx, cy, nx, ny, th1, s);
}
}  // namespace msdd

// ---- which memory the device holds -----------------------------------------
static std::vector<std::pair<const void *, size_t>> g_foreign;   // arrays that are not the device's, and their bytes
static std::vector<std::pair<const void *, size_t>> g_asked;
namespace msdd_rt {
bool device_holds(int device, const void *p, size_t bytes)
{
    g_asked.emplace_back(p, bytes);
    for (auto &f : g_foreign)
        if (f.first == p) return false;
    return device == 0;
}
}  // namespace msdd_rt

// ---- a small problem --------------------------------------------------------
struct Problem {
    int n;
    std::vector<double> rho, x, y, b;
    explicit Problem(int n_) : n(n_), rho((size_t)n_ * n_, 1.0), x(rho.size()), y(rho.size())
    {
        for (int j = 0; j < n; ++j)
            for (int i = 0; i < n; ++i) {
                x[(size_t)j * n + i] = i / (n - 1.0);
                y[(size_t)j * n + i] = j / (n - 1.0);
            }
        for (int s = 0; s < 4; ++s)
            for (int c = 0; c < 2; ++c)
                for (int k = 0; k < n; ++k) {
                    const double t = k / (n - 1.0), at[2] = {s < 2 ? (double)s : t, s < 2 ? t : s - 2.0};
                    b.push_back(at[c]);
                }
        x[0] = 0.0;
    }
};

static mesh_sdd_desc make_desc(int n, int sub, int precision, int K, uint32_t id = 0)
{
    mesh_sdd_desc d;
    std::memset(&d, 0, sizeof d);
    d.struct_size = sizeof d;
    d.n_xi = d.n_eta = n;
    d.sub_xi = d.sub_eta = sub;
    d.K = K;
    d.Lx = d.Ly = 1.0;
    d.tau = 0.01;
    d.precision = precision;
    d.bridge = 1;
    d.instance_id = id;
    return d;
}

static mesh_sdd_step make_step(const Problem &p, int64_t N, int on_device)
{
    mesh_sdd_step s;
    std::memset(&s, 0, sizeof s);
    s.struct_size = sizeof s;
    s.inputs_on_device = on_device;
    s.x_cur = p.x.data();
    s.y_cur = p.y.data();
    s.bnd_t0 = s.bnd_t1 = p.b.data();
    s.paths_per_node = N;
    return s;
}

struct Out {
    std::vector<double> a[5];
    mesh_sdd_result r;
    explicit Out(int m, int on_device)
    {
        std::memset(&r, 0, sizeof r);
        r.struct_size = sizeof r;
        r.outputs_on_device = on_device;
        for (auto &v : a) v.assign((size_t)m, -1.0);
        double **p[5] = {&r.mean_x, &r.mean_y, &r.se_x, &r.se_y, &r.exit_frac};
        for (int k = 0; k < 5; ++k) *p[k] = a[k].data();
    }
};

struct Fixture {
    mesh_sdd_ctx *ctx = nullptr;
    std::vector<mesh_sdd *> h;
    Fixture(size_t budget = 0) { check(mesh_sdd_ctx_create(0, budget, nullptr, &ctx) == MESH_SDD_OK, "ctx_create"); }
    ~Fixture()
    {
        for (mesh_sdd *i : h) check(mesh_sdd_destroy(i) == MESH_SDD_OK, "destroy");
        check(mesh_sdd_ctx_destroy(ctx) == MESH_SDD_OK, "ctx_destroy");
    }
    mesh_sdd *add(const Problem &p, const mesh_sdd_desc &d)
    {
        mesh_sdd *i = nullptr;
        check(mesh_sdd_create(ctx, &d, &i) == MESH_SDD_OK, "create");
        check(mesh_sdd_set_monitor(i, p.rho.data(), 0) == MESH_SDD_OK, "set_monitor");
        h.push_back(i);
        return i;
    }
};

// ---------------------------------------------------------------------------
static void scenario_arrays()
{
    Problem p(17);
    p.x[0] = 0.25;   // recognised in the staged copy
    for (int precision : {MESH_SDD_FP32, MESH_SDD_FP64}) {
        Fixture f;
        mesh_sdd *h = f.add(p, make_desc(17, 2, precision, 20));
        const int m = mesh_sdd_num_interface_nodes(h);
        const size_t n = p.x.size() * 8, nb = p.b.size() * 8;
        for (bool noalloc : {false, true}) {
            auto solve = noalloc ? mesh_sdd_solve_interfaces_noalloc : mesh_sdd_solve_interfaces;
            mesh_sdd_step st = make_step(p, 300, 1);
            Out o(m, 1);
            // the device's own arrays: used where they are, each asked for its whole length
            g_foreign.clear();
            g_asked.clear();
            check(solve(h, &st, &o.r) == MESH_SDD_OK, "solve");
            check(g_prep_x == p.x.data(), "the mesh is read in place");
            check(g_final[0] == o.a[0].data(), "the results are written in place");
            for (auto &want : {std::make_pair((const void *)p.x.data(), n), std::make_pair((const void *)p.y.data(), n),
                               std::make_pair((const void *)p.b.data(), nb),
                               std::make_pair((const void *)o.a[4].data(), (size_t)m * 8)}) {
                bool found = false;
                for (auto &a : g_asked) found = found || a == want;
                check(found, "an array of %zu bytes was not looked up", want.second);
            }
            // each input in turn not the device's: a staged copy of the same values
            for (const double *bad : {p.x.data(), p.y.data(), p.b.data()}) {
                g_foreign.assign(1, {bad, 0});
                check(solve(h, &st, &o.r) == MESH_SDD_OK, "solve with a foreign input");
                check(g_prep_x != p.x.data() && g_prep_first == 0.25, "a foreign input is read in place");
                check(g_final[0] == o.a[0].data(), "the results are written in place");
            }
            // each result in turn not the device's: copied out
            for (int k = 0; k < 5; ++k) {
                Out q(m, 1);
                g_foreign.assign(1, {q.a[k].data(), 0});
                check(solve(h, &st, &q.r) == MESH_SDD_OK, "solve with a foreign result");
                check(g_prep_x == p.x.data(), "the mesh is read in place");
                check(g_final[k] != q.a[k].data() && q.a[k][0] == 0.0 && q.a[k][m - 1] == 0.0,
                      "foreign result %d: written in place, or not at all", k);
            }
        }
        // a batch: the other request still writes in place
        mesh_sdd *both[2] = {h, h};
        mesh_sdd_step st[2] = {make_step(p, 300, 1), make_step(p, 300, 1)};
        Out a(m, 1), b(m, 1);
        mesh_sdd_result res[2] = {a.r, b.r};
        g_foreign.assign(1, {a.a[2].data(), 0});
        check(mesh_sdd_solve_batch(both, st, res, 2, nullptr) == MESH_SDD_OK, "batch");
        check(g_final[0] == b.a[0].data() && a.a[0][0] == 0.0, "batch with a foreign result");
        g_foreign.clear();
    }
}

// ---------------------------------------------------------------------------
// Requests of 29 nodes at N = 1280 on 8 CUs: 10 chunks of 128 paths per node,
// or 20 slices whose records take 29 * 20 * 528 bytes.
static const int64_t kN = 1280;
static const size_t kRecords = 29 * 20 * sizeof(msdd::SliceRec);

static uint64_t in_use(mesh_sdd_ctx *ctx)
{
    mesh_sdd_stats st;
    std::memset(&st, 0, sizeof st);
    st.struct_size = sizeof st;
    check(mesh_sdd_ctx_stats(ctx, &st) == MESH_SDD_OK, "stats");
    return st.hbm_in_use;
}

// Submits one request per instance, all of them queued before the first is
// staged, and waits for all; the most memory in use and requests running.
static void serve(Fixture &f, const Problem &p, size_t count, uint64_t *most, uint64_t *running)
{
    g_slices.clear();
    g_most_in_use = g_most_running = 0;
    g_watched = f.ctx;
    std::vector<mesh_sdd_ticket> t(count);
    mesh_sdd_step st = make_step(p, kN, 0);
    {
        std::lock_guard<std::mutex> hold(g_gate);
        for (size_t k = 0; k < count; ++k) check(mesh_sdd_submit(f.h[k], &st, &t[k]) == MESH_SDD_OK, "submit");
    }
    Out o(29, 0);
    for (size_t k = 0; k < count; ++k) check(mesh_sdd_wait(f.ctx, t[k], &o.r, -1) == MESH_SDD_OK, "wait");
    g_watched = nullptr;
    if (most) *most = g_most_in_use;
    if (running) *running = g_most_running;
}

static size_t sliced()
{
    size_t n = 0;
    for (uint32_t s : g_slices) n += s != 0;
    return n;
}

static void scenario_budget()
{
    Problem p(17), big(65);
    size_t tables, tables65, base;
    uint64_t most = 0, running = 0;
    {
        // the cost of an instance's tables and of a request in whole chunks
        // (paths of fewer than 64 substeps never run in slices)
        Fixture f;
        f.add(p, make_desc(17, 2, MESH_SDD_FP32, 20));
        tables = in_use(f.ctx);
        serve(f, p, 1, &most, nullptr);
        base = most - tables;
        check(in_use(f.ctx) == tables, "a finished request leaves nothing in use");
        f.add(big, make_desc(65, 2, MESH_SDD_FP32, 20));
        tables65 = in_use(f.ctx) - tables;
        check(base > 10000 && base < kRecords / 2, "base %zu", base);
    }
    {
        // room for everything: slices, alone, in a batch and served
        Fixture f;
        for (int k = 0; k < 5; ++k) f.add(p, make_desc(17, 2, MESH_SDD_FP32, 100, k));
        serve(f, p, 5, &most, &running);
        check(g_slices.size() == 5 && sliced() == 5, "%zu of 5 requests in slices", sliced());
        check(running >= 3, "%d requests ran together", (int)running);
        check(most == 5 * tables + running * (base + kRecords), "%zu bytes in use", (size_t)most);
        check(in_use(f.ctx) == 5 * tables, "finished requests leave nothing in use");
    }
    {
        // room for the requests in whole chunks beside each other and for
        // the records of one: they run together, as whole chunks
        Fixture f(5 * tables + 5 * base + kRecords);
        for (int k = 0; k < 5; ++k) f.add(p, make_desc(17, 2, MESH_SDD_FP32, 100, k));
        serve(f, p, 5, &most, &running);
        check(running >= 3, "%d requests ran together", (int)running);
        check(most <= 5 * tables + 5 * base + kRecords, "%zu bytes in use of %zu", (size_t)most,
              5 * tables + 5 * base + kRecords);
    }
    {
        // resident tables leave room for one request in whole chunks only
        const size_t budget = tables + 4 * tables65 + base + kRecords / 2;
        check(budget > base + kRecords, "the records alone would fit the budget");
        Fixture f(budget);
        f.add(p, make_desc(17, 2, MESH_SDD_FP32, 100));
        for (int k = 0; k < 4; ++k) f.add(big, make_desc(65, 2, MESH_SDD_FP32, 100, 1 + k));
        serve(f, p, 1, &most, &running);
        check(most <= budget && sliced() == 0, "%zu bytes in use of %zu", (size_t)most, budget);
        g_slices.clear();
        mesh_sdd_step st = make_step(p, kN, 0);
        Out o(29, 0);
        check(mesh_sdd_solve_interfaces(f.h[0], &st, &o.r) == MESH_SDD_OK && sliced() == 0, "a blocking solve");
    }
    {
        // a batch: slices for as many of its requests as the budget has room for
        Fixture f(5 * tables + 5 * base + 2 * kRecords + kRecords / 2);
        std::vector<mesh_sdd_step> st(5, make_step(p, kN, 0));
        std::vector<Out> o(5, Out(29, 0));
        std::vector<mesh_sdd_result> r;
        for (int k = 0; k < 5; ++k) {
            f.add(p, make_desc(17, 2, MESH_SDD_FP32, 100, k));
            o[k] = Out(29, 0);
            r.push_back(o[k].r);
        }
        g_slices.clear();
        check(mesh_sdd_solve_batch(f.h.data(), st.data(), r.data(), 5, nullptr) == MESH_SDD_OK, "batch");
        check(g_slices.size() == 5 && sliced() == 2, "%zu of 5 requests in slices", sliced());
        g_slices.clear();
        mesh_sdd_step dev = make_step(p, kN, 1);
        Out d(29, 1);
        check(mesh_sdd_solve_interfaces_noalloc(f.h[0], &dev, &d.r) == MESH_SDD_OK && sliced() == 1,
              "the no-allocation solve's records lie in its own scratch");
    }
}

// ---------------------------------------------------------------------------
static void scenario_fp64()
{
    // 29 nodes at N = 6400: 100 items of 64 paths per node, or 25 of 256
    Problem p(17);
    const size_t n = 17 * 17, np = 19 * 19, nb = 8 * 17;
    const size_t large = 2 * n * 8 + 2 * np * 12 + 2 * nb * 12 + 29 * (25 * sizeof(msdd::Partial) + sizeof(msdd::NodeSpan)) +
                         29 * 5 * 8 + sizeof(msdd::InstView) + 64;
    const size_t small = large + 29 * 75 * sizeof(msdd::Partial);
    size_t tables = 0;
    auto run = [&](size_t budget, uint32_t items, size_t bytes) {
        Fixture f(budget);
        f.add(p, make_desc(17, 2, MESH_SDD_FP64, 20));
        tables = in_use(f.ctx);
        g_most_in_use = 0;
        g_watched = f.ctx;
        mesh_sdd_step st = make_step(p, 6400, 0);
        mesh_sdd_ticket t = 0;
        Out o(29, 0);
        check(mesh_sdd_submit(f.h[0], &st, &t) == MESH_SDD_OK, "submit within a budget of %zu", budget);
        check(mesh_sdd_wait(f.ctx, t, &o.r, -1) == MESH_SDD_OK, "wait");
        check(g_items == items, "%u items per node", g_items);
        check(g_most_in_use == tables + bytes, "%zu bytes charged, %zu allocated", (size_t)g_most_in_use - tables, bytes);
        g_watched = nullptr;
        // the blocking and the no-allocation solve have the same sums
        check(mesh_sdd_solve_interfaces(f.h[0], &st, &o.r) == MESH_SDD_OK && g_items == items, "solve");
        mesh_sdd_step dev = make_step(p, 6400, 1);
        Out d(29, 1);
        check(mesh_sdd_solve_interfaces_noalloc(f.h[0], &dev, &d.r) == MESH_SDD_OK && g_items == items, "noalloc");
    };
    run(0, 100, small);
    run(16 * (small - large), 100, small);
    run(16 * (small - large) - 16, 25, large);
    run(large, 25, large);   // what a request of 256-path items always fitted
    Fixture f(large - 1);
    f.add(p, make_desc(17, 2, MESH_SDD_FP64, 20));
    mesh_sdd_step st = make_step(p, 6400, 0);
    mesh_sdd_ticket t = 0;
    check(mesh_sdd_submit(f.h[0], &st, &t) == MESH_SDD_E_BUDGET, "a request past the budget");
}

// ---------------------------------------------------------------------------
static void scenario_boxes()
{
    // every subdomain of at most 4096 interior and 1024 boundary nodes
    // (subdomain_fits_lds) has a workgroup with a thread for each boundary
    // node and threads for all interior ones
    long boxes = 0;
    for (int px = 2; px <= 511; ++px)
        for (int py = 2; py <= 511; ++py) {
            const long nin = (long)(px - 1) * (py - 1), nb = 2L * (px + 1) + 2L * (py - 1);
            if (nin > (long)msdd::kSubBlock * msdd::kSubPerThread || nb > msdd::kSubBlock) continue;
            ++boxes;
            for (bool exact : {false, true}) {
                if (exact && !msdd::power_of_two(px)) continue;   // they divide a power of two
                if (exact && !msdd::power_of_two(py)) continue;
                const msdd::SubShape h = msdd::subdomain_shape(px, py, exact);
                const long per = h.nodes, segs = per ? (long)(px - 1) * ((py - 1 + per - 1) / per) : 0;
                check(h.block >= 64 && h.block <= msdd::kSubBlock && h.block % 64 == 0 && h.inner <= h.block && per <= 4 &&
                          (exact ? per <= py - 1 && segs <= h.inner : per * h.inner >= nin) && h.first_bnd >= 0 &&
                          h.first_bnd + nb <= h.block && (h.first_bnd >= h.inner || h.block == msdd::kSubBlock),
                      "%d x %d cells: %d nodes on %d threads, boundary from %d, block %d", px, py, h.nodes, h.inner,
                      h.first_bnd, h.block);
            }
        }
    check(boxes > 10000, "%ld boxes", boxes);
    // forced on boxes of 3 x 500 cells, by themselves the tiles'
    Fixture f;
    mesh_sdd_desc d = make_desc(0, 1, MESH_SDD_FP64, 1);
    d.n_xi = 13;
    d.n_eta = 501;
    d.sub_xi = 4;
    d.tau = 1e-6;
    const std::vector<double> a((size_t)13 * 501, 1.0), b(4 * 514, 1.0);
    std::vector<double> x(a), y(a);
    mesh_sdd *h = nullptr;
    check(mesh_sdd_create(f.ctx, &d, &h) == MESH_SDD_OK, "create");
    f.h.push_back(h);
    check(mesh_sdd_set_monitor(h, a.data(), 0) == MESH_SDD_OK, "set_monitor");
    for (int solver : {1, 2}) {
        mesh_sdd_mp_opts o;
        std::memset(&o, 0, sizeof o);
        o.struct_size = sizeof o;
        o.solver = solver;
        g_lds_solves = g_sweeps = 0;
        check(mesh_sdd_subdomain_solve(h, a.data(), a.data(), b.data(), a.data(), a.data(), x.data(), y.data(), &o, 0) ==
                  MESH_SDD_OK, "solver %d", solver);
        check((g_lds_solves == 1) == (solver == 1) && (g_sweeps > 0) == (solver == 2), "solver %d: %d LDS solves, %d sweeps",
              solver, g_lds_solves, g_sweeps);
    }
}

// ---------------------------------------------------------------------------
// Every item of every range in exactly one job, no job empty, queues in order.
static void check_jobs(const char *what)
{
    std::vector<std::vector<int>> seen;
    for (const msdd::WorkRange &w : g_ranges) seen.emplace_back(w.count, 0);
    for (const msdd::WinJob &j : g_jobs) {
        check(j.count > 0, "%s: an empty job", what);
        const msdd::WorkRange &w = g_ranges[j.range];
        for (uint32_t k = 0; k < j.count; ++k) {
            const uint32_t q = j.q0 + k - w.first;
            if (q < w.count) ++seen[j.range][q];
            else check(false, "%s: item %u outside its range", what, q);
        }
    }
    for (auto &r : seen)
        for (int c : r)
            if (c != 1) return check(false, "%s: an item in %d jobs", what, c);
    check(g_queues.b[0] == 0 && g_queues.b[msdd::kJobQueues] == g_jobs.size(), "%s: queues", what);
}

static void scenario_jobs()
{
    // 8 workgroups of 16 waves; 161^2 in 8 x 8: 2177 nodes in 3 x 3 blocks
    Fixture f;
    Problem p(161), q(193);
    mesh_sdd *h = f.add(p, make_desc(161, 8, MESH_SDD_FP32, 100, 1));
    mesh_sdd *g = f.add(q, make_desc(193, 2, MESH_SDD_FP32, 100, 2));
    mesh_sdd *k = f.add(q, make_desc(193, 2, MESH_SDD_FP32, 20, 3));   // short paths
    auto run = [&](mesh_sdd *i, const Problem &pr, int64_t n, uint32_t stride) {
        mesh_sdd_step st = make_step(pr, n, 0);
        st.interface_stride = stride;
        Out o(mesh_sdd_num_interface_nodes(i), 0);
        g_jobs.clear();
        check(mesh_sdd_solve_interfaces(i, &st, &o.r) == MESH_SDD_OK, "solve");
        return g_jobs.size();
    };
    struct {
        mesh_sdd *i;
        const Problem *p;
        int64_t n;
        uint32_t stride;
        size_t jobs;   // at most (or one for each block); 0: not of equal size
    } cases[] = {{g, &q, 64, 0, 8},    {g, &q, 65, 0, 8},   {g, &q, 150, 0, 16}, {g, &q, 640, 0, 24},
                 {g, &q, 1300, 0, 0},  {h, &p, 64, 0, 16},  {h, &p, 200, 0, 0},  {h, &p, 100, 4, 9},
                 {h, &p, 1, 0, 16},    {k, &q, 640, 0, 0},  {g, &q, 1, 8, 8}};
    for (auto &c : cases) {
        const size_t n = run(c.i, *c.p, c.n, c.stride);
        check_jobs("alone");
        if (!c.jobs) continue;
        check(n <= c.jobs, "N = %d: %zu jobs, at most %zu", (int)c.n, n, c.jobs);
        for (size_t a = 1; a < g_jobs.size(); ++a)   // the jobs of a block differ by one item at most
            if (g_jobs[a].i0 == g_jobs[a - 1].i0 && g_jobs[a].j0 == g_jobs[a - 1].j0)
                check(std::abs((int)g_jobs[a].count - (int)g_jobs[a - 1].count) <= 1, "N = %d: jobs of %u and %u items",
                      (int)c.n, g_jobs[a].count, g_jobs[a - 1].count);
    }
    // several instances, and a job_split that is set
    std::vector<mesh_sdd *> all{h, g, k};
    std::vector<mesh_sdd_step> st{make_step(p, 500, 0), make_step(q, 64, 0), make_step(q, 900, 0)};
    std::vector<Out> o;
    std::vector<mesh_sdd_result> r;
    for (mesh_sdd *i : all) o.emplace_back(mesh_sdd_num_interface_nodes(i), 0);
    for (auto &x : o) r.push_back(x.r);
    for (int split : {0, 1, 4096}) {
        mesh_sdd_launch l;
        std::memset(&l, 0, sizeof l);
        l.struct_size = sizeof l;
        l.job_split = split;
        check(mesh_sdd_set_launch(f.ctx, &l) == MESH_SDD_OK, "set_launch");
        g_jobs.clear();
        check(mesh_sdd_solve_batch(all.data(), st.data(), r.data(), 3, nullptr) == MESH_SDD_OK, "batch");
        check(g_ranges.size() == 3, "three ranges");
        check_jobs("batch");
        run(g, q, 1300, 0);
        check_jobs("split");
        run(g, q, 150, 0);
        check_jobs("split, few items");
    }
    // the no-allocation solve: the same jobs where its scratch has room for the list
    check(mesh_sdd_set_launch(f.ctx, nullptr) == MESH_SDD_OK, "set_launch");
    const size_t alone = run(g, q, 640, 0);
    mesh_sdd_step dev = make_step(q, 640, 1);
    Out d(mesh_sdd_num_interface_nodes(g), 1);
    g_jobs.clear();
    check(mesh_sdd_solve_interfaces_noalloc(g, &dev, &d.r) == MESH_SDD_OK, "noalloc");
    check_jobs("noalloc");
    check(g_jobs.size() == alone, "noalloc: %zu jobs, %zu", g_jobs.size(), alone);
}

// ---------------------------------------------------------------------------
static void scenario_slices()
{
    // 381 nodes on 8 CUs: more slices than waves
    Fixture f;
    Problem q(193);
    mesh_sdd *g = f.add(q, make_desc(193, 2, MESH_SDD_FP32, 100, 2));
    Out o(mesh_sdd_num_interface_nodes(g), 0);
    for (auto &c : std::vector<std::pair<int64_t, bool>>{{64, true}, {65, false}, {95, false}, {96, true}, {130, true}}) {
        g_slices.clear();
        mesh_sdd_step st = make_step(q, c.first, 0);
        check(mesh_sdd_solve_interfaces(g, &st, &o.r) == MESH_SDD_OK, "solve");
        check((sliced() == 1) == c.second, "N = %d", (int)c.first);
    }
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "arrays")
        scenario_arrays();
    else if (what == "budget")
        scenario_budget();
    else if (what == "boxes")
        scenario_boxes();
    else if (what == "jobs")
        scenario_jobs();
    else if (what == "slices")
        scenario_slices();
    else if (what == "fp64")
        scenario_fp64();
    else {
        std::fprintf(stderr, "unknown scenario %s\n", what.c_str());
        return 2;
    }
    if (g_failures) {
        std::fprintf(stderr, "%d check(s) failed\n", g_failures);
        return 1;
    }
    std::printf("%s: all checks passed\n", what.c_str());
    return 0;
}
