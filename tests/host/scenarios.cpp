// Scenarios of the library's host code on the stand-in runtime: one per run,
// named by the first argument; the exit status says whether it held.
#include <chrono>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include <unistd.h>

#include <hip/hip_runtime.h>

#include "../../include/stag.h"
#include "hip_stub.h"

using hipstub::ctl;

static int failures = 0;
#define CHECK(c)                                                    \
    do {                                                            \
        if (!(c)) {                                                 \
            ++failures;                                             \
            fprintf(stderr, "line %d: %s does not hold\n", __LINE__, #c); \
        }                                                           \
    } while (0)

struct Lattice {
    int L[4];
    size_t vh() const { return (size_t)L[0] * L[1] * L[2] * L[3] / 2; }
};

static stag_gauge* make_gauge(stag_ctx* c, const Lattice& l, int mask) {
    std::vector<double> U(l.vh() * 2 * 72, 0.0);
    stag_gauge* g = nullptr;
    CHECK(stag_gauge_create(c, l.L, U.data(), 0, mask, &g) == STAG_OK);
    return g;
}

static stag_field* make_field(stag_ctx* c, stag_gauge* g, int prec, int n, int parity = 0) {
    stag_field* f = nullptr;
    CHECK(stag_field_create(c, g, parity, prec, n, &f) == STAG_OK);
    return f;
}

struct Solve {
    int prec = STAG_F32, n = 1, use_graph = 1, small = 1;
    hipStream_t stream = nullptr;
};

static int solve(stag_ctx* c, stag_gauge* g, const Solve& s) {
    stag_field *b = make_field(c, g, STAG_F64, s.n), *x = make_field(c, g, STAG_F64, s.n);
    std::vector<double> mass(s.n, 0.1);
    std::vector<stag_cg_stats> st(s.n);
    stag_cg_params p;
    stag_cg_params_default(&p);
    p.inner_prec = s.prec;
    p.use_graph = s.use_graph;
    p.small_lattice = s.small;
    const int rc = stag_cg_solve(c, g, mass.data(), b, x, &p, st.data(), s.stream);
    if (rc == STAG_OK)
        for (auto& t : st) CHECK(t.status == STAG_OK && t.true_rel_res == 0.0);
    stag_field_destroy(b);
    stag_field_destroy(x);
    return rc;
}

static const Lattice k44{{4, 4, 4, 4}}, k66{{6, 6, 6, 6}}, k88{{8, 8, 8, 8}}, k16{{16, 16, 16, 16}};

static void wait_ticket(stag_ctx* c, stag_ticket t) {
    while (stag_solver_poll(c, t, nullptr, nullptr, nullptr) == STAG_PENDING)
        std::this_thread::sleep_for(std::chrono::microseconds(200));
}

// Nothing is destroyed before the runtime has retired its work: solves of
// every group pattern, a change of the launch shapes (which drops the graphs),
// gauges and contexts destroyed right after, serving batches released.
static void lifetime() {
    for (int n : {1, 3, 5, 8, 11, 16}) {
        stag_ctx* c = nullptr;
        CHECK(stag_create(0, 0, &c) == STAG_OK);
        stag_gauge* g = make_gauge(c, k88, STAG_MASK_F64 | STAG_MASK_F32);
        hipStream_t own = nullptr;
        (void)hipStreamCreateWithFlags(&own, 0);
        stag_field *b = make_field(c, g, STAG_F64, n), *x = make_field(c, g, STAG_F64, n);
        std::vector<double> mass(n, 0.1), v(k88.vh() * 6 * n, 1.0);
        stag_cg_params p;
        stag_cg_params_default(&p);
        p.inner_prec = STAG_F32;
        p.small_lattice = 0;
        CHECK(stag_cg_solve(c, g, mass.data(), b, x, &p, nullptr, own) == STAG_OK);
        stag_tune_cfg t;
        CHECK(stag_tune_get(c, STAG_F32, n, (int64_t)k88.vh(), &t) == STAG_OK);
        CHECK(stag_tune_set(c, STAG_F32, n, (int64_t)k88.vh(), &t) == STAG_OK);
        CHECK(stag_cg_solve(c, g, mass.data(), b, x, &p, nullptr, own) == STAG_OK);
        stag_gauge_destroy(g);
        g = make_gauge(c, k88, STAG_MASK_F64 | STAG_MASK_F32);
        stag_ticket id = 0;
        CHECK(stag_solver_submit(c, g, 0.1, n, v.data(), 1e-8, STAG_F32, &id) == STAG_OK);
        wait_ticket(c, id);
        CHECK(stag_gauge_destroy(g) == STAG_OK);
        stag_destroy(c);
        (void)hipStreamSynchronize(own);
        (void)hipStreamDestroy(own);
    }
}

// A solve that ends with a launch error leaves nothing of its own running.
static void launch_error() {
    for (int at : {1, 2, 3, 4}) {
        stag_ctx* c = nullptr;
        CHECK(stag_create(0, 0, &c) == STAG_OK);
        stag_gauge* g = make_gauge(c, k88, STAG_MASK_F64 | STAG_MASK_F32);
        stag_field *b = make_field(c, g, STAG_F64, 8), *x = make_field(c, g, STAG_F64, 8);
        std::vector<double> mass(8, 0.1);
        stag_cg_params p;
        stag_cg_params_default(&p);
        p.inner_prec = STAG_F32;
        p.small_lattice = 0;
        ctl.fail_graph_launch = at;
        CHECK(stag_cg_solve(c, g, mass.data(), b, x, &p, nullptr, nullptr) == STAG_EDEVICE);
        CHECK(hipstub::in_flight() == 0);
        ctl.fail_graph_launch = 0;
        CHECK(stag_cg_solve(c, g, mass.data(), b, x, &p, nullptr, nullptr) == STAG_OK);
        stag_destroy(c);
    }
}

// Which kernels a solve took.
struct Path {
    int persist, tiny;
};
static Path path_of(const Lattice& l, const Solve& s) {
    stag_ctx* c = nullptr;
    CHECK(stag_create(0, 0, &c) == STAG_OK);
    stag_gauge* g = make_gauge(c, l, STAG_MASK_F64 | STAG_MASK_F32 | STAG_MASK_F16S);
    const int p0 = ctl.persist, t0 = ctl.tiny;
    CHECK(solve(c, g, s) == STAG_OK);
    const Path r{ctl.persist - p0, ctl.tiny - t0};
    stag_destroy(c);
    return r;
}

// Lattices of up to 648 sites per parity are solved inside a kernel whether
// graphs are asked for or not.
static void small_without_graphs() {
    for (const Lattice& l : {k44, k66})
        for (int prec : {STAG_F64, STAG_F32, STAG_F16S})
            for (int n : {1, 4, 16})
                for (int graph : {0, 1}) {
                    Solve s;
                    s.prec = prec;
                    s.n = n;
                    s.use_graph = graph;
                    const Path p = path_of(l, s);
                    CHECK(p.persist + p.tiny > 0);
                    s.use_graph = 1 - graph;
                    const Path q = path_of(l, s);
                    CHECK((p.persist > 0) == (q.persist > 0) && (p.tiny > 0) == (q.tiny > 0));
                    s.small = 0;
                    const Path r = path_of(l, s);
                    CHECK(r.persist + r.tiny == 0);
                }
    Solve s;
    s.use_graph = 0;
    CHECK(path_of(k88, s).persist == 0);
}

// What solves a lattice of up to 128 sites per parity does not depend on how many
// right-hand sides the call has (the two solvers add their sums in another order).
static void small_same_for_blocks() {
    for (const Lattice& l : {Lattice{{2, 2, 2, 2}}, Lattice{{4, 4, 4, 2}}, k44})
        for (int prec : {STAG_F64, STAG_F32, STAG_F16S}) {
            Solve s;
            s.prec = prec;
            const Path one = path_of(l, s);
            for (int n : {2, 5, 16}) {
                s.n = n;
                const Path p = path_of(l, s);
                CHECK((p.tiny > 0) == (one.tiny > 0) && (p.persist > 0) == (one.persist > 0));
            }
        }
}

// The budget covers the memory kept from destroyed objects too: it is never
// exceeded, kept memory is given back before an object is refused, and a block
// used again comes back as a new one would (fields zero).
static void budget() {
    const size_t budget = 24u << 20;
    stag_ctx* c = nullptr;
    CHECK(stag_create(0, budget, &c) == STAG_OK);
    auto held = [&] {
        size_t b = 0;
        CHECK(stag_memory_used(c, &b) == STAG_OK);
        CHECK(b == ctl.malloc_held && b <= budget);
        return b;
    };
    const Lattice sizes[] = {k88, {{8, 8, 8, 4}}, {{8, 8, 8, 12}}, {{8, 8, 4, 12}}, {{8, 8, 8, 16}}};
    for (int k = 0; k < 25; ++k) {
        const Lattice l = sizes[k % 5];
        std::vector<double> U(l.vh() * 2 * 72, 0.0);
        stag_gauge* g = nullptr;
        CHECK(stag_gauge_create(c, l.L, U.data(), 1, STAG_MASK_F64 | STAG_MASK_F32, &g) == STAG_OK);
        const int n = 1 + k % 3;
        stag_field* f = make_field(c, g, STAG_F64, n);
        std::vector<double> v(l.vh() * 6 * n, 1.0);
        CHECK(stag_field_export(f, v.data(), 0, nullptr) == STAG_OK);
        for (double x : v)
            if (x != 0.0) {
                CHECK(x == 0.0);
                break;
            }
        v.assign(v.size(), 3.0);
        CHECK(stag_field_import(f, v.data(), 0, nullptr) == STAG_OK);
        Solve s;
        s.n = 1;
        CHECK(solve(c, g, s) == STAG_OK);
        held();
        stag_field_destroy(f);
        CHECK(stag_gauge_destroy(g) == STAG_OK);
        held();
    }
    CHECK(ctl.malloc_peak <= budget);
    // an object larger than what is left is refused, one that fits once the kept
    // memory is given back is not
    stag_gauge *g = nullptr, *g2 = nullptr;
    const Lattice big{{16, 16, 16, 8}}, most{{8, 8, 8, 26}};
    std::vector<double> U(big.vh() * 2 * 72, 0.0);
    CHECK(stag_gauge_create(c, big.L, U.data(), 1, STAG_MASK_F64, &g) == STAG_ENOMEM);
    CHECK(stag_gauge_create(c, most.L, U.data(), 1, STAG_MASK_F64 | STAG_MASK_F32, &g2) == STAG_OK);
    CHECK(held() > budget * 9 / 10);
    stag_destroy(c);
    CHECK(ctl.malloc_held == 0);
}

// A device synchronisation that fails has not waited: what is destroyed then is
// not handed out again while kernels may still use it.
static void failed_sync() {
    stag_ctx* c = nullptr;
    CHECK(stag_create(0, 0, &c) == STAG_OK);
    hipStream_t own = nullptr;
    (void)hipStreamCreateWithFlags(&own, 0);
    stag_gauge* g = make_gauge(c, k44, STAG_MASK_F64);
    stag_field *a = make_field(c, g, STAG_F64, 1), *b = make_field(c, g, STAG_F64, 1);
    const double m = 0.1;
    ctl.kernel_ms = 100;
    for (int k = 0; k < 2; ++k) {
        CHECK(stag_apply_A(c, g, &m, a, b, own) == STAG_OK);
        ctl.fail_device_sync = 1;
        if (k == 0) {
            stag_field_destroy(b);
            b = make_field(c, g, STAG_F64, 1);
        } else {
            CHECK(stag_gauge_destroy(g) == STAG_OK);
            g = make_gauge(c, k44, STAG_MASK_F64);
        }
        CHECK(hipstub::in_flight() == 0);
        ctl.fail_device_sync = 0;
    }
    ctl.kernel_ms = 0;
    stag_destroy(c);
    CHECK(ctl.malloc_held == 0);
}

// Temporaries of the operator calls and host copies get the memory kept from
// destroyed objects when the device has no other left.
static void temporaries() {
    stag_ctx* c = nullptr;
    CHECK(stag_create(0, 0, &c) == STAG_OK);
    stag_gauge* g = make_gauge(c, k88, STAG_MASK_F64);
    stag_field *a = make_field(c, g, STAG_F64, 1), *b = make_field(c, g, STAG_F64, 1);
    std::vector<double> v(k88.vh() * 6, 1.0);
    const double m = 0.1;
    for (int call = 0; call < 3; ++call) {
        // kept memory: a gauge and its fields; then only a few KB more
        stag_gauge* h = make_gauge(c, k66, STAG_MASK_F64);
        CHECK(stag_gauge_destroy(h) == STAG_OK);
        ctl.memory_limit = ctl.held + 4096;
        if (call == 0) CHECK(stag_field_import(a, v.data(), 0, nullptr) == STAG_OK);
        if (call == 1) CHECK(stag_field_export(a, v.data(), 0, nullptr) == STAG_OK);
        if (call == 2) CHECK(stag_apply_A(c, g, &m, a, b, nullptr) == STAG_OK);
        (void)hipDeviceSynchronize();
        ctl.memory_limit = 0;
    }
    stag_destroy(c);
}

// A resident kernel whose waits run out: the solve starts over with a kernel per
// stage (from its guess too), and later solves of the context do not try again
// until they are told to.
static void resident_gives_up() {
    for (int n : {1, 3}) {
        stag_ctx* c = nullptr;
        CHECK(stag_create(0, 0, &c) == STAG_OK);
        stag_gauge* g = make_gauge(c, k88, STAG_MASK_F64 | STAG_MASK_F32);
        Solve s;
        s.n = n;
        int64_t solves = 0, gave_up = 0;
        CHECK(solve(c, g, s) == STAG_OK);
        CHECK(stag_resident_counts(c, &solves, &gave_up) == STAG_OK && solves == 1 && gave_up == 0);
        CHECK(stag_resident_wait(c, -1.0) == STAG_OK);
        const int stages = ctl.stage;
        CHECK(solve(c, g, s) == STAG_OK);
        CHECK(ctl.stage > stages);
        CHECK(stag_resident_counts(c, &solves, &gave_up) == STAG_OK && solves == 2 && gave_up == 1);
        const int launched = ctl.persist;
        for (int prec : {STAG_F32, STAG_F64}) {
            s.prec = prec;
            CHECK(solve(c, g, s) == STAG_OK);
        }
        CHECK(ctl.persist == launched);
        CHECK(stag_resident_wait(c, 2.0) == STAG_OK);
        CHECK(solve(c, g, s) == STAG_OK);
        CHECK(ctl.persist > launched);
        CHECK(stag_resident_counts(c, &solves, &gave_up) == STAG_OK && solves == 3 && gave_up == 1);
        stag_destroy(c);
    }
}

// Solves of several threads at once, each with a context of its own: small ones
// run in resident kernels beside each other, never with more workgroups than 7/8
// of one XCD's units; a large one runs alone or with a kernel per stage.
static void resident_together() {
    ctl.kernel_ms = 20;
    auto run = [](const Lattice& l, int threads, int64_t* resident) {
        std::vector<std::thread> th;
        std::atomic<int64_t> sum{0};
        for (int k = 0; k < threads; ++k)
            th.emplace_back([&] {
                stag_ctx* c = nullptr;
                CHECK(stag_create(0, 0, &c) == STAG_OK);
                stag_gauge* g = make_gauge(c, l, STAG_MASK_F64);
                Solve s;
                s.prec = STAG_F64;
                for (int i = 0; i < 3; ++i) CHECK(solve(c, g, s) == STAG_OK);
                int64_t n = 0, gave_up = 0;
                CHECK(stag_resident_counts(c, &n, &gave_up) == STAG_OK && gave_up == 0);
                sum += n;
                stag_destroy(c);
            });
        for (auto& t : th) t.join();
        *resident = sum;
    };
    int64_t n = 0;
    run(k44, 6, &n);  // 2 workgroups each
    CHECK(n == 18 && ctl.persist_most >= 2 && ctl.blocks_most <= 28);
    ctl.persist_most = ctl.blocks_most = 0;
    run(k66, 6, &n);  // 11 each: two at a time
    CHECK(n >= 3 && ctl.persist_most <= 2 && ctl.blocks_most <= 28);
    ctl.persist_most = ctl.blocks_most = 0;
    run(k16, 3, &n);  // 256: alone
    CHECK(n >= 1 && ctl.persist_most == 1);
    ctl.kernel_ms = 0;
}

// A resident kernel that holds more than 7/8 of an XCD's compute units (in fp32
// 128 sites a workgroup; up to 32 of them on one XCD, more over all) leaves them
// after a bounded number of iterations.
static void resident_launches_are_short() {
    const struct {
        Lattice l;
        int n;
        bool is_short;
    } cases[] = {{k16, 1, true},  {{{16, 16, 16, 32}}, 1, true}, {{{8, 8, 8, 16}}, 1, true},
                 {k88, 16, true}, {{{8, 8, 8, 12}}, 1, false},   {k88, 8, false}};
    for (auto& k : cases) {
        stag_ctx* c = nullptr;
        CHECK(stag_create(0, 0, &c) == STAG_OK);
        stag_gauge* g = make_gauge(c, k.l, STAG_MASK_F64 | STAG_MASK_F32);
        ctl.persist_iters = 0;
        Solve s;
        s.n = k.n;
        CHECK(solve(c, g, s) == STAG_OK);
        CHECK(ctl.persist_iters > 0 && (ctl.persist_iters <= 64) == k.is_short);
        stag_destroy(c);
    }
}

// stag_tune covers the kernels that the iterations run: groups of 8, 4 and the
// rest, not only the whole block.
static void tuned_sizes() {
    char path[] = "/tmp/stag_tune_XXXXXX";
    const int fd = mkstemp(path);
    CHECK(fd >= 0);
    setenv("STAG_TUNE_CACHE", path, 1);
    const std::vector<std::pair<int, std::set<int>>> want = {
        {1, {1}}, {4, {4}}, {6, {4, 8}}, {8, {4, 8}}, {11, {3, 4, 12}}, {12, {4, 12}}, {13, {1, 4, 8, 16}}, {16, {8, 16}}};
    for (auto& w : want) {
        CHECK(truncate(path, 0) == 0);
        stag_ctx* c = nullptr;
        CHECK(stag_create(0, 0, &c) == STAG_OK);
        stag_gauge* g = make_gauge(c, k88, STAG_MASK_F64 | STAG_MASK_F32);
        for (int again = 0; again < 2; ++again)
            CHECK(stag_tune(c, g, STAG_F32, w.first, nullptr, nullptr) == STAG_OK);
        int loaded = 0, measured = 0;
        CHECK(stag_tune_counts(c, &loaded, &measured) == STAG_OK && loaded == 1 && measured == 1);
        std::set<int> got;
        FILE* f = fopen(path, "r");
        char arch[64];
        int pairs, r12, prec, n;
        unsigned vh;
        char rest[128];
        while (f && fscanf(f, "%63s %d %d %u %d %d :%127[^\n]", arch, &pairs, &r12, &vh, &prec, &n, rest) == 7) got.insert(n);
        if (f) fclose(f);
        CHECK(got == w.second);
        double us[3];
        CHECK(stag_time_kernels(c, g, STAG_F32, w.first, 2, us) == STAG_OK);
        stag_destroy(c);
    }
    close(fd);
    unlink(path);
}

// 12-parameter links that are not SU(3) are refused as that, with memory for the
// copies or without, and leave nothing held; good ones without memory ENOMEM.
static void bad_links() {
    for (int mask : {STAG_MASK_F64, STAG_MASK_F16S, STAG_MASK_F64 | STAG_MASK_F32 | STAG_MASK_F16S})
        for (size_t budget : {(size_t)0, (size_t)65536, (size_t)1 << 20})
            for (int bad : {0, 1}) {
                ctl.bad_links = bad;
                stag_ctx* c = nullptr;
                CHECK(stag_create(0, budget, &c) == STAG_OK);
                std::vector<double> U(k88.vh() * 2 * 72, 0.0);
                stag_gauge* g = nullptr;
                const int rc = stag_gauge_create(c, k88.L, U.data(), 0, mask | STAG_GAUGE_R12, &g);
                CHECK(rc == (bad ? STAG_EINVAL : budget == 0 || (mask == STAG_MASK_F16S && budget > 900000) ? STAG_OK : STAG_ENOMEM));
                CHECK((g != nullptr) == (rc == STAG_OK));
                stag_destroy(c);
                CHECK(ctl.malloc_held == 0);
            }
    ctl.bad_links = 0;
}

// The groups of a block run on streams of different hardware queues, whatever
// streams the program created before; streams taken while none were found to are
// not kept for the next gauge.
static void groups_on_queues_of_their_own() {
    ctl.paired_queues = 1;
    for (int before = 0; before < 4; ++before)
        for (int n : {5, 8, 11, 13, 16}) {
            hipStream_t other = nullptr;
            for (int k = 0; k < before; ++k) (void)hipStreamCreateWithFlags(&other, 0);
            stag_ctx* c = nullptr;
            CHECK(stag_create(0, 0, &c) == STAG_OK);
            for (int gauge = 0; gauge < 2; ++gauge) {
                stag_gauge* g = make_gauge(c, k88, STAG_MASK_F64 | STAG_MASK_F32);
                ctl.queues_used = 0;
                Solve s;
                s.n = n;
                s.small = 0;
                CHECK(solve(c, g, s) == STAG_OK);
                CHECK(__builtin_popcount(ctl.queues_used) == (n == 11 || n == 13 ? 3 : 2));
                CHECK(stag_gauge_destroy(g) == STAG_OK);
            }
            stag_destroy(c);
            CHECK(ctl.malloc_held == 0);
        }
    for (int before = 0; before < 4; ++before)
        for (int n : {8, 13}) {
            hipStream_t other = nullptr;
            for (int k = 0; k < before; ++k) (void)hipStreamCreateWithFlags(&other, 0);
            stag_ctx* c = nullptr;
            CHECK(stag_create(0, 0, &c) == STAG_OK);
            for (int busy : {1, 0}) {
                ctl.never_apart = busy;
                stag_gauge* g = make_gauge(c, k88, STAG_MASK_F64 | STAG_MASK_F32);
                ctl.queues_used = 0;
                Solve s;
                s.n = n;
                s.small = 0;
                CHECK(solve(c, g, s) == STAG_OK);
                CHECK(busy || __builtin_popcount(ctl.queues_used) == (n == 13 ? 3 : 2));
                CHECK(stag_gauge_destroy(g) == STAG_OK);
            }
            stag_destroy(c);
            CHECK(ctl.malloc_held == 0);
        }
}

int main(int argc, char** argv) {
    static const std::map<std::string, std::function<void()>> all = {
        {"lifetime", lifetime},
        {"launch_error", launch_error},
        {"budget", budget},
        {"failed_sync", failed_sync},
        {"temporaries", temporaries},
        {"tuned_sizes", tuned_sizes},
        {"bad_links", bad_links},
        {"groups_on_queues_of_their_own", groups_on_queues_of_their_own},
        {"resident_gives_up", resident_gives_up},
        {"resident_together", resident_together},
        {"resident_launches_are_short", resident_launches_are_short},
        {"small_same_for_blocks", small_same_for_blocks},
        {"small_without_graphs", small_without_graphs},
    };
    auto it = argc > 1 ? all.find(argv[1]) : all.end();
    if (it == all.end()) return 2;
    it->second();
    fflush(nullptr);
    _Exit(failures || hipstub::violations() ? 1 : 0);
}
