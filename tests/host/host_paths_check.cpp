// Checks of the library's host code on a device that is the host (fake_device.h):
// what it enqueues, in which order and where, what it waits for, and what it does
// when a call fails.  The argument names the check; exit status 0 when it holds.
#include "fake_device.h"

// the code under test, with its file-scope state in reach
#include "da_api.cpp"

namespace dapt {
void logged_build(const std::vector<double> &temps, HostTables &ht) {
    (void)fake::note("build_host_tables");
    build_host_tables(temps, ht);
}
}  // namespace dapt
#define build_host_tables logged_build
#include "da_server.cpp"
#undef build_host_tables

#include <cstdio>

static long g_bad = 0;
#define CHECK(c)                                              \
    do {                                                      \
        if (!(c)) {                                           \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c); \
            ++g_bad;                                          \
        }                                                     \
    } while (0)

// Q of N variables: +-1 couplings, or (wide) up to 300 in size, times scale.
static std::vector<int32_t> instance(int N, bool wide = false, int32_t scale = 1) {
    std::vector<int32_t> Q((size_t)N * N, 0);
    uint32_t r = 12345u + (uint32_t)N;
    for (int i = 0; i < N; ++i)
        for (int j = i; j < N; ++j) {
            r = r * 1664525u + 1013904223u;
            const int32_t v = wide ? (int32_t)((r >> 8) % 601u) - 300 : ((r >> 8) & 1u ? 1 : -1);
            Q[(size_t)i * N + j] = v * scale;
        }
    return Q;
}
static da_ctx *create(int N, bool wide = false, int32_t scale = 1, int32_t hint = 0) {
    da_ctx *c = nullptr;
    const std::vector<int32_t> Q = instance(N, wide, scale);
    if (da_create(Q.data(), N, hint, &c) != DA_OK) std::printf("da_create(%d) failed\n", N), ++g_bad;
    return c;
}
static da_schedule schedule(double T_hi = 30.0, double T_lo = 1.0, int32_t levels = 8) {
    da_schedule s{};
    s.T_hi = T_hi;
    s.T_lo = T_lo;
    s.kind = DA_SCHED_GEOMETRIC;
    s.n_levels = levels;
    s.eoff_inc = 1;
    s.init = DA_INIT_ZEROS;
    s.trial = DA_TRIAL_PARALLEL;
    return s;
}
struct Batch {
    std::vector<da_batch_item> items;
    void add(da_ctx *c, int32_t replicas = 3, int64_t steps = 100) {
        da_batch_item it{};
        it.ctx = c;
        it.schedule = schedule();
        it.replicas = replicas;
        it.steps = steps;
        it.seed = items.size() + 1;
        items.push_back(it);
    }
    int run() { return da_anneal_batch(items.data(), (int32_t)items.size(), nullptr); }
    ~Batch() {
        for (auto &it : items) da_destroy(it.ctx);
    }
};
static bool is_launch(const fake::Call &c) { return c.name == "mix" || c.name == "hipGraphLaunch"; }

// A launch of a batch fails: the call returns only when everything it enqueued
// before is done (the kernels read tables that the next call rewrites).
static void batch_error() {
    Batch b;
    b.add(create(40));
    b.add(create(40, true));
    b.add(create(40, true, 0, 4));
    CHECK(b.run() == DA_OK);
    for (int ok = 0; ok < 3; ++ok) {   // launches that go out before one fails
        fake::reset();
        fake::st().fail_from["mix"] = ok;
        CHECK(b.run() != DA_OK);
        const auto &log = fake::st().log;
        for (size_t q = 0; q < log.size(); ++q) {
            if (!is_launch(log[q])) continue;
            bool waited = false;
            for (size_t w = q + 1; w < log.size(); ++w)
                waited = waited || log[w].name == "hipDeviceSynchronize" ||
                         (log[w].name == "hipStreamSynchronize" && log[w].stream == log[q].stream);
            CHECK(waited);
        }
    }
    fake::reset();
    CHECK(b.run() == DA_OK);
}

// Jobs of the wave kernels and of the table-driven kernel in one batch: launched
// side by side, without a wait on the host between, and joined to one stream.
static void batch_overlap() {
    Batch b;
    b.add(create(40));
    b.add(create(41, true, 1, 2));
    b.add(create(60, false, 1, DA_STORE_SPARSE));
    b.add(create(42, false, 1 << 16, 2));      // its factor is past 16 bits
    fake::reset();
    CHECK(b.run() == DA_OK);
    CHECK(fake::count("mix") == 2 && fake::count("hipGraphLaunch") == 1);
    const auto &log = fake::st().log;
    std::vector<size_t> at;
    for (size_t q = 0; q < log.size(); ++q)
        if (is_launch(log[q])) at.push_back(q);
    for (size_t q = at.front(); q < at.back(); ++q)
        CHECK(log[q].name != "hipStreamSynchronize" && log[q].name != "hipDeviceSynchronize");
    const void *s = nullptr;   // the caller's stream: the outputs leave on it
    size_t out = log.size();
    for (size_t q = 0; q < log.size(); ++q)
        if (log[q].name == "outputs" && out == log.size()) s = log[out = q].stream;
    for (size_t q : at) {
        for (size_t r : at) CHECK(q == r || log[q].stream != log[r].stream);
        if (log[q].stream == s) continue;
        const void *ev = nullptr;   // recorded behind the launch, waited for on s
        for (size_t w = q + 1; w < out && !ev; ++w)
            if (log[w].name == "hipEventRecord" && log[w].stream == log[q].stream) ev = log[w].event;
        bool joined = false;
        for (size_t w = q + 1; w < out; ++w)
            joined = joined || (log[w].name == "hipStreamWaitEvent" && log[w].stream == s &&
                                log[w].event == ev);
        CHECK(ev && joined);
    }
}

// More items than the tables hold: chunk by chunk, each after the one before.
static void batch_chunks() {
    Batch b;
    const int32_t R = 1200000;
    b.add(create(1), R);
    b.add(create(1, false, 1, DA_STORE_SPARSE), R);
    fake::reset();
    CHECK(b.run() == DA_OK);
    const size_t per_item = 4;   // replicas of N = 1 per item of the mixed launches
    size_t items = 0;
    for (int n : fake::st().mix_blocks) {
        CHECK(n <= BatchRunner::kCapItems);
        items += (size_t)n;
    }
    CHECK(items == (R + per_item - 1) / per_item);
    // (16 replicas per item of the persistent launches)
    CHECK(fake::count("hipGraphLaunch") ==
          (R / 16 + BatchRunner::kCapItems - 1) / BatchRunner::kCapItems);
    const auto &log = fake::st().log;
    for (size_t q = 0; q < log.size(); ++q) {
        if (!is_launch(log[q])) continue;
        bool waited = false;   // before a table is written again
        for (size_t w = q + 1; w < log.size(); ++w) {
            waited = waited || log[w].name == "hipStreamSynchronize";
            CHECK(waited || log[w].name != "hipMemcpyAsync");
        }
    }
}

// da_last_kernel_stats after a batch states the launch each job went in: that of
// its descriptor, in a batch that fits the chip and in one that fills it.
static void batch_stats() {
    for (int32_t many : {3, 40000}) {
        Batch b;
        b.add(create(40), many);
        b.add(create(100, true, 1, 2));
        b.add(create(700), 5);
        b.add(create(3000), 2);
        b.add(create(60, false, 1, DA_STORE_SPARSE));
        for (auto &it : b.items)   // (a batch is timed on its first context only)
            CHECK(da_anneal_async(it.ctx, &it.schedule, 0, 1, 10, 1, nullptr, nullptr, nullptr) ==
                  DA_OK);
        fake::reset();
        CHECK(b.run() == DA_OK);
        for (auto &it : b.items) {
            da_kernel_stats st{};
            CHECK(da_last_kernel_stats(it.ctx, &st) == DA_OK);
            bool found = false;
            size_t launch = 0;
            for (const JobDesc &J : fake::st().mix_jobs) {
                if (J.seed != it.seed) continue;
                found = true;
                CHECK(st.flips_per_lane == J.F && st.rng_waves == J.NH && st.w_in_lds == J.w_lds);
                CHECK(st.replicas_per_block == J.RPW && st.threads == 512 && st.draw_estimates == 1);
                for (int n : fake::st().mix_blocks) launch += st.blocks == n ? 1 : 0;
                CHECK(launch > 0 && st.blocks >= (it.replicas + J.RPW - 1) / J.RPW);
            }
            if (!found) CHECK(st.flips_per_lane == 8 && st.threads == 1024 && st.blocks == 256);
            CHECK(found == (it.ctx->ell_D == 0));
        }
    }
}

// da_create waits for its own work only: no call that waits for the device.
static void create_waits() {
    for (int N : {100, 300}) {
        fake::reset();
        da_ctx *c = create(N);
        CHECK(fake::count("hipFree") == 0 && fake::count("hipDeviceSynchronize") == 0);
        const size_t held = fake::st().used;
        da_destroy(c);
        CHECK(held >= (size_t)N * N && held < 2 * (size_t)N * N + 65536 && fake::st().used == 0);
    }
}

// Where da_create derives an instance: up to 224 variables the host is faster.
static void create_sizes() {
    for (int N : {1, 129, 200, 224, 225, 256, 700}) {
        fake::reset();
        da_destroy(create(N));
        CHECK(fake::count("derive") == (N > 224 ? 1 : 0));
    }
}

// da_create where the image fits but not the upload buffer, alone or beside it:
// the same instance, and no error left for the next call's launches.
static void create_memory() {
    const int N = 300, ld = 320;
    const std::vector<int32_t> Q = instance(N, true);
    const size_t image = (size_t)ld * ld * 2 + ld * 4;
    for (size_t room : {image, (size_t)N * N * 4 + derive_scratch_bytes(N) + 60000}) {
        fake::reset();
        fake::st().memory = fake::st().used + room;
        da_ctx *c = nullptr;
        CHECK(da_create(Q.data(), N, 0, &c) == DA_OK);
        fake::st().memory = SIZE_MAX;
        if (!c) continue;
        CHECK(c->dtype == 2 && c->wscale == 1);
        const int16_t *W = static_cast<const int16_t *>(c->d_W);
        for (int i = 0; i < ld; ++i)
            for (int j = 0; j < ld; ++j) {
                const int32_t w = i < N && j < N && i != j
                                      ? Q[(size_t)i * N + j] + Q[(size_t)j * N + i] : 0;
                CHECK(W[(size_t)i * ld + j] == w);
            }
        for (int i = 0; i < N; ++i) CHECK(c->d_b[i] == Q[(size_t)i * N + i]);
        const da_schedule s = schedule();
        CHECK(da_anneal_async(c, &s, 0, 1, 10, 1, nullptr, nullptr, nullptr) == DA_OK);
        da_destroy(c);
    }
    // not even the image fits
    fake::reset();
    fake::st().memory = fake::st().used + image / 2;
    da_ctx *c = nullptr;
    CHECK(da_create(Q.data(), N, 0, &c) == DA_ENOMEM && c == nullptr);
    fake::st().memory = SIZE_MAX;
}

// Outputs of an anneal or of tempering on their way to the host, more than a
// pinned block holds: whole, with and without device memory to spare, and with no
// device memory kept that da_get_info leaves out, nor a wait for the device.
static void outputs_memory() {
    const int N = 300, R = 3000;
    std::vector<uint8_t> bx((size_t)R * N), x((size_t)R * N);
    std::vector<int64_t> bE(R), E(R), n(R);
    const da_result all{bx.data(), bE.data(), x.data(), E.data(), n.data()};
    da_ctx *c = create(N);
    const da_schedule s = schedule();
    auto no_outputs = [&] {
        return da_anneal_async(c, &s, 0, R, 10, 1, nullptr, nullptr, nullptr);
    };
    CHECK(no_outputs() == DA_OK);   // state and tables are there
    const double T[2] = {1.0, 2.0};
    auto whole = [&] {
        for (int r = 0; r < R; ++r) {
            CHECK(E[r] == 3 * r && bE[r] == -r && n[r] == 7 * r);
            for (int i = 0; i < N; ++i)
                if (x[(size_t)r * N + i] != (r + i) % 3 || bx[(size_t)r * N + i] != (r ^ i) % 5)
                    ++g_bad;
        }
    };
    auto held = [&] {
        da_info info{};
        CHECK(da_get_info(c, &info) == DA_OK);
        return fake::st().used - (size_t)info.device_bytes;
    };
    const size_t before = held();
    for (bool room : {false, true}) {
        fake::reset();
        if (!room) fake::st().memory = fake::st().used;
        CHECK(da_anneal(c, &s, R, 10, 1, const_cast<da_result *>(&all)) == DA_OK);
        whole();
        CHECK(held() == before);
        CHECK(fake::count("hipFree") == 0 && fake::count("hipDeviceSynchronize") == 0);
        CHECK((fake::count("hipMemcpy2DAsync") == 0) == room);
        CHECK(no_outputs() == DA_OK);   // no error left behind
    }
    da_pt_result pt{};
    pt.best_x = bx.data();
    pt.best_E = bE.data();
    pt.final_x = x.data();
    pt.final_E = E.data();
    pt.n_accept = n.data();
    fake::reset();
    CHECK(da_pt(c, T, 2, R / 2, 2, 5, 0, 1, &pt) == DA_OK);
    whole();
    fake::st().memory = fake::st().used;   // the buffers of tempering are there
    CHECK(da_pt(c, T, 2, R / 2, 2, 5, 0, 1, &pt) == DA_OK);
    whole();
    CHECK(fake::count("hipMemcpy2DAsync") == 0);
    da_destroy(c);
    fake::st().memory = SIZE_MAX;
}

// Small outputs where pinned memory cannot be had, and where the wait for the
// kernel that writes it fails (it may still write then).
static void outputs_pinned() {
    const int N = 70, R = 5;
    std::vector<uint8_t> bx(N * R), x(N * R);
    std::vector<int64_t> bE(R), E(R), n(R);
    da_result all{bx.data(), bE.data(), x.data(), E.data(), n.data()};
    da_ctx *c = create(N);
    const da_schedule s = schedule();
    CHECK(da_anneal_async(c, &s, 0, R, 10, 1, nullptr, nullptr, nullptr) == DA_OK);
    fake::reset();
    fake::st().fail_from["hipHostMalloc"] = 0;
    CHECK(da_anneal(c, &s, R, 10, 1, &all) == DA_OK);
    CHECK(E[R - 1] == 3 * (R - 1) && x[N + 1] == 2 && bx[N + 1] == 0);
    fake::reset();
    CHECK(da_anneal(c, &s, R, 10, 1, &all) == DA_OK);
    CHECK(fake::count("hipHostMalloc") == 1);
    fake::reset();
    fake::st().fail_from["hipStreamSynchronize"] = 0;
    CHECK(da_anneal(c, &s, R, 10, 1, &all) == DA_EDEVICE);
    fake::reset();
    CHECK(da_anneal(c, &s, R, 10, 1, &all) == DA_OK);
    CHECK(fake::count("hipHostMalloc") == 1);   // another block
    da_destroy(c);
}

// A call fails for want of memory, with that error; the next one succeeds.
static void error_once() {
    const std::vector<int32_t> Q = instance(70);
    da_ctx *c = create(70);
    const da_schedule s = schedule();
    for (int R : {40, 80}) {   // the tables' memory, then more state
        fake::reset();
        fake::st().fail_from["hipMalloc"] = 0;
        CHECK(da_anneal_async(c, &s, 0, R, 10, 1, nullptr, nullptr, nullptr) == DA_ENOMEM);
        fake::st().fail_from.clear();
        CHECK(da_anneal_async(c, &s, 0, R, 10, 1, nullptr, nullptr, nullptr) == DA_OK);
    }
    da_ctx *d = nullptr;
    fake::reset();
    fake::st().fail_from["hipMalloc"] = 0;
    CHECK(da_create(Q.data(), 70, 0, &d) == DA_ENOMEM);
    fake::st().fail_from.clear();
    CHECK(da_anneal_async(c, &s, 0, 4, 10, 1, nullptr, nullptr, nullptr) == DA_OK);
    da_destroy(c);
}

// The server builds the level tables of the jobs that need them on its preparation
// threads, not on the device worker, and hands them on; the others' not at all.
static void server_tables() {
    for (bool wide : {false, true}) {   // (wide: a factor past the wave kernels' range)
        const int N = 60, R = 4;
        const std::vector<int32_t> Q = instance(N, false, wide ? 1 << 16 : 1);
        fake::reset();
        da_server *srv = nullptr;
        CHECK(da_server_create(size_t(1) << 30, nullptr, &srv) == DA_OK);
        da_job job{};
        job.Q = Q.data();
        job.N = N;
        job.dtype_hint = 2;
        job.schedule = schedule(wide ? 4e6 : 30.0, wide ? 1e5 : 1.0);
        job.replicas = R;
        job.steps = 1000;
        job.seed = 1;
        uint64_t ticket = 0;
        CHECK(da_submit(srv, &job, &ticket) == DA_OK);
        da_job_stats st{};
        CHECK(da_wait(srv, ticket, nullptr, &st) == DA_OK);
        da_server_destroy(srv);
        std::thread::id built, launched;
        for (const auto &c : fake::st().log) {
            if (c.name == "build_host_tables") built = c.thread;
            if (is_launch(c)) launched = c.thread;
        }
        CHECK(fake::count("hipGraphLaunch") == (wide ? 1 : 0) && fake::count("mix") == (wide ? 0 : 1));
        CHECK(fake::count("build_host_tables") == (wide ? 1 : 0));
        CHECK(built != launched && launched != std::thread::id());
    }
    // tables made before are taken as they are, and only for their temperatures
    const std::vector<double> temps = {5.0, 2.5};
    HostTables ht;
    build_host_tables(temps, ht);
    ht.thr[7] += 1;
    std::string err;
    auto lt = get_level_tables(temps, err, &ht);
    CHECK(lt && lt->d_thr[7] == ht.thr[7] && lt->L == 2);
    auto other = get_level_tables({5.0, 2.25}, err, &ht);
    CHECK(other && other->d_thr[7] == ht.thr[7] - 1);
}

// Temperature lists leave the cache with the contexts that held them.
static void temps_bounded() {
    da_ctx *c = create(40), *d = create(41);
    const da_schedule keep = schedule(20.0, 1.5);
    CHECK(da_anneal_async(d, &keep, 0, 1, 10, 1, nullptr, nullptr, nullptr) == DA_OK);
    for (int q = 0; q < 300; ++q) {
        const da_schedule s = schedule(30.0 + q, 1.0, 4 + q % 9);
        CHECK(da_anneal_async(c, &s, 0, 1, 10, 1, nullptr, nullptr, nullptr) == DA_OK);
        CHECK(g_temps.size() <= 3);
    }
    const int lists = fake::count("hipMalloc");
    CHECK(da_anneal_async(c, &keep, 0, 1, 10, 1, nullptr, nullptr, nullptr) == DA_OK);
    CHECK(fake::count("hipMalloc") == lists);   // d's list is still there
    da_destroy(c);
    da_destroy(d);
}

// Launch shapes of the table-driven kernel are timed, also for short schedules, on
// windows that stay inside the schedule, once for a size and replica count.
static void tuner_windows() {
    for (int N : {71, 93, 111, 133})
        for (bool sparse : {true, false}) {
            da_ctx *c = sparse ? create(N, true, 1, DA_STORE_SPARSE) : create(N + 1, false, 1 << 15, 2);
            int32_t R = 1;   // (a new bucket of replica counts each time)
            for (int64_t S : {65, 100, 575, 2000}) {
                R *= 2;
                const da_schedule s = schedule(2e5, 1e4, 128);
                fake::reset();
                CHECK(da_anneal_async(c, &s, 0, R, S, 1, nullptr, nullptr, nullptr) == DA_OK);
                const auto &runs = fake::st().runs;
                CHECK(runs.size() > 1 && fake::count("wave") == 0);
                for (const JobDesc &J : runs)
                    CHECK(J.s0 >= 0 && J.s0 <= J.s1 && J.s1 <= J.S && J.S == S);
                CHECK(runs.back().s0 == 0 && runs.back().s1 == S);
                const size_t timed = runs.size();
                fake::reset();
                CHECK(da_anneal_async(c, &s, 0, R, S, 1, nullptr, nullptr, nullptr) == DA_OK);
                CHECK(fake::st().runs.size() == 1 && timed > 2);
            }
            da_destroy(c);
        }
}

// Not a check: the step kernels that wave_shape chooses over sizes, couplings and
// replicas, one a line: type, flips per lane, then W in LDS, or waves and Philox
// blocks of a team as the launcher tells its variants apart.
static void list_shapes() {
    std::map<std::string, int> seen;
    std::vector<int> sizes;
    for (int N = 1; N <= 8192; N += N < 700 ? 1 : N < 4200 ? 13 : 61) sizes.push_back(N);
    for (int N : {1024, 1025, 2048, 2049, 4096, 4097, 8192}) sizes.push_back(N);
    for (int N : sizes)
        for (int dtype : {1, 2, 4})
            for (int per_cu : {1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 17, 40}) {
                da_ctx c;
                c.N = N;
                c.ld = (N + 63) / 64 * 64;
                c.dtype = dtype;
                c.hbound = 1000;
                LaunchShape sh;
                CHECK(wave_shape(&c, 256 * per_cu, 1.0, 30.0, sh));
                char line[80];
                const char type = dtype == 1 ? 'a' : dtype == 2 ? 's' : 'i';
                if (sh.NW > 1)
                    std::snprintf(line, sizeof line, "team %c %d %d %d", type, sh.F,
                                  sh.NW <= 2 ? 2 : sh.NW <= 4 ? 4 : 16,
                                  sh.NH == 0 ? 0 : sh.NH * 512 >= N ? 1 : 2);
                else
                    std::snprintf(line, sizeof line, "wave %c %d %d", type, sh.F, sh.w_lds);
                seen[line] = 1;
            }
    for (auto &s : seen) std::printf("%s\n", s.first.c_str());
}

int main(int argc, char **argv) {
    const std::map<std::string, void (*)()> checks = {
        {"batch_error", batch_error},
        {"batch_overlap", batch_overlap},
        {"batch_chunks", batch_chunks},
        {"batch_stats", batch_stats},
        {"create_waits", create_waits},
        {"create_sizes", create_sizes},
        {"create_memory", create_memory},
        {"outputs_memory", outputs_memory},
        {"outputs_pinned", outputs_pinned},
        {"error_once", error_once},
        {"server_tables", server_tables},
        {"temps_bounded", temps_bounded},
        {"tuner_windows", tuner_windows},
        {"list_shapes", list_shapes},
    };
    auto it = argc > 1 ? checks.find(argv[1]) : checks.end();
    if (it == checks.end()) return 2;
    it->second();
    std::printf("failures %ld\n", g_bad);
    return g_bad ? 1 : 0;
}
