// da_api.cpp -- the C ABI of include/da.h: contexts, anneals, parallel
// tempering and energies on one gfx950 device.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <vector>

#include "da_runtime.h"

using namespace dapt;

namespace dapt {

namespace {
thread_local std::string t_err;
constexpr size_t kEventPool = 1024;

int64_t gcd64(int64_t a, int64_t b) {
    a = a < 0 ? -a : a;
    b = b < 0 ? -b : b;
    while (b) {
        const int64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}
}  // namespace

void set_thread_error(const std::string &msg) { t_err = msg; }

int fail(da_ctx *ctx, int code, const std::string &msg) {
    if (ctx) ctx->err = msg;
    t_err = msg;
    // reported here: the thread's next launch is not to find it again
    if (code == DA_ENOMEM || code == DA_EDEVICE) (void)hipGetLastError();
    return code;
}

int check_hip(da_ctx *ctx, hipError_t e, const char *what) {
    if (e == hipSuccess) return DA_OK;
    std::string msg = std::string(what) + ": " + hipGetErrorString(e);
    return fail(ctx, e == hipErrorOutOfMemory ? DA_ENOMEM : DA_EDEVICE, msg);
}

void StateBuf::release() {
    if (h) (void)hipFree(h);   // the start of the one allocation
    h = nullptr; x = bx = nullptr; E = bE = nacc = nullptr; eoff = nullptr;
    cap = 0;
}

int64_t StateBuf::bytes_for(int32_t R, int32_t ld) {
    return (int64_t)R * ld * (4 + 1 + 1) + (int64_t)R * (8 * 3 + 4);
}

int64_t StateBuf::bytes() const { return bytes_for(cap, ld); }

bool StateBuf::ensure(int32_t R, int32_t ld_, std::string &err) {
    if (R <= cap && ld_ == ld) return true;
    release();
    ld = ld_;
    const int32_t n = std::max(R, 1);
    const size_t rows = (size_t)n * ld;   // (ld: a multiple of 64, so all parts are aligned)
    char *p = nullptr;
    if (hipMalloc(&p, (size_t)bytes_for(n, ld)) != hipSuccess) {
        err = "out of device memory for replica state";
        return false;
    }
    h = reinterpret_cast<int32_t *>(p);
    x = reinterpret_cast<uint8_t *>(h + rows);
    bx = x + rows;
    E = reinterpret_cast<int64_t *>(bx + rows);
    bE = E + n;
    nacc = bE + n;
    eoff = reinterpret_cast<int32_t *>(nacc + n);
    cap = n;
    return true;
}

int validate_schedule(const da_schedule *s, std::string &err) {
    if (!s) {
        err = "schedule is null";
        return DA_EINVAL;
    }
    if (s->kind != DA_SCHED_GEOMETRIC && s->kind != DA_SCHED_LINEAR_BETA) {
        err = "unknown schedule kind";
        return DA_EINVAL;
    }
    if (s->n_levels < 0 || s->n_levels > kMaxLevels) {
        err = "n_levels must be in [0, 4096] (0: a new temperature every step)";
        return DA_EINVAL;
    }
    if (s->eoff_inc < 0) {
        err = "eoff_inc must be >= 0";
        return DA_EINVAL;
    }
    if (s->init != DA_INIT_ZEROS && s->init != DA_INIT_RANDOM) {
        err = "unknown init";
        return DA_EINVAL;
    }
    if ((s->trial != DA_TRIAL_PARALLEL && s->trial != DA_TRIAL_SINGLE) || s->reserved != 0) {
        err = "trial must be DA_TRIAL_PARALLEL or DA_TRIAL_SINGLE, reserved 0";
        return DA_EINVAL;
    }
    const bool zero = (s->T_hi == 0.0 && s->T_lo == 0.0);
    if (!zero && !(s->T_hi > 0.0 && s->T_lo > 0.0 && std::isfinite(s->T_hi) &&
                   std::isfinite(s->T_lo))) {
        err = "temperatures must be finite and > 0 (or both 0)";
        return DA_EINVAL;
    }
    return DA_OK;
}

// Launch shape: F variables per lane, NW = ceil(N / 64F) waves per replica,
// RPW replicas per workgroup.  W goes to LDS when small (it then serves every
// row fetch at LDS latency).
LaunchShape choose_shape(const da_ctx *ctx, int32_t R, const da_launch *launch,
                         bool anneal_mode, bool direct) {
    LaunchShape sh;
    int stage = anneal_mode ? 1 : 0;
    const int cus = ctx->cus;
    // Few replicas per CU: each replica's step latency is the limit, so spread
    // a replica over more waves (4 variables per lane) and move the random
    // numbers to their own waves.  A full chip is limited by total work: 8
    // variables per lane and lazy draws.
    const bool latency_bound = R <= 2 * cus;
    const int want_help = launch ? launch->rng_waves : 0;
    bool help = want_help > 0 || (want_help == 0 && latency_bound);
    sh.F = (launch && launch->flips_per_lane) ? launch->flips_per_lane : (latency_bound ? 4 : 8);
    if (sh.F != 2 && sh.F != 4 && sh.F != 8) sh.F = 8;
    if (sh.F == 2 && ctx->dtype > 2) sh.F = 4;   // two per lane: 8/16-bit couplings only
    sh.NW = (ctx->N + 64 * sh.F - 1) / (64 * sh.F);
    if (sh.NW > 16) {  // keep a replica within one workgroup (N <= 8192)
        sh.F = 8;
        sh.NW = (ctx->N + 64 * sh.F - 1) / (64 * sh.F);
    }
    const int nblk = (ctx->N + 7) / 8;
    sh.NH = help ? (nblk + 63) / 64 : 0;
    if (sh.NW + sh.NH > 16) sh.NH = 0;
    const int per = sh.NW + sh.NH;
    int rpw = (launch && launch->replicas_per_block) ? launch->replicas_per_block : 1;
    rpw = std::max(1, std::min(rpw, 16 / per));
    rpw = std::min(rpw, std::max(R, 1));
    sh.RPW = rpw;
    // parallel tempering with one replica per workgroup stages the level of
    // that replica for each round (the launcher picks that variant)
    if (!anneal_mode && rpw == 1) stage = 1;
    // what an anneal may stage in LDS: the sparse lists, else dense W
    const int64_t w_bytes = (anneal_mode && ctx->ell_D > 0)
                                ? (int64_t)ctx->N * ctx->ell_D * 4
                                : (int64_t)ctx->N * ctx->ld * ctx->dtype;
    const int want = launch ? launch->w_in_lds : 0;
    const bool sparse = anneal_mode && ctx->ell_D > 0;
    // dense W goes to LDS automatically only when small; row lists whenever they fit
    sh.w_lds = (want >= 0 && w_bytes <= ((want > 0 || sparse) ? device_lds_limit() : 32 * 1024))
                   ? 1
                   : 0;
    sh.threads = 64 * per * sh.RPW;
    sh.blocks = (R + sh.RPW - 1) / sh.RPW;
    // direct tables (narrow bands) are staged too when the schedule has them;
    // W gives way to them, and they give way when even that does not fit
    // (sparse row lists take a kernel variant without them)
    sh.direct = anneal_mode && direct && !sparse ? 1 : 0;
    const size_t limit = (size_t)device_lds_limit();
    sh.lds = run_lds_bytes(sh.NW, sh.RPW, sh.F, sh.w_lds ? (int)w_bytes : 0, stage, sh.NH, sparse,
                           sh.direct);
    if (sh.lds > limit && sh.w_lds) {
        sh.w_lds = 0;
        sh.lds = run_lds_bytes(sh.NW, sh.RPW, sh.F, 0, stage, sh.NH, sparse, sh.direct);
    }
    if (sh.lds > limit && sh.direct) {
        sh.direct = 0;
        sh.lds = run_lds_bytes(sh.NW, sh.RPW, sh.F, 0, stage, sh.NH, sparse);
    }
    // per-draw estimates (handed over by random-number waves, or evaluated by
    // the compute lanes under lazy draws): a multi-wave replica reading W from
    // global memory (the wide variants), 4 or 8 flips per lane, and fields
    // small enough for the estimate path's int32 sums; not with direct tables
    // Left to choose (no tuner), estimates only where fields span many coupling
    // units: a cost then rarely falls inside an estimate's window of a few
    // units, while +-1-like instances meet it every step or two.
    const int want_gen = launch ? launch->draw_estimates : 0;
    const bool wide16 = ctx->dtype != 2 || (ctx->wscale < (1 << 15) && ctx->wscale > -(1 << 15));
    const bool fine_fields = ctx->hbound >= 4096 * (int64_t)std::abs(ctx->wscale);
    if ((want_gen > 0 || (want_gen == 0 && fine_fields)) && anneal_mode && !sparse &&
        !sh.direct && !sh.w_lds && sh.NW > 1 && sh.F >= 4 && wide16 &&
        ctx->hbound <= kGenFieldMax) {
        const size_t lg = run_lds_bytes(sh.NW, sh.RPW, sh.F, 0, stage, sh.NH, false, false, true);
        if (lg <= limit) {
            sh.gen = 1;
            sh.lds = lg;
        }
    }
    return sh;
}

JobDesc make_job(const da_ctx *ctx, const LevelTables *lt, int32_t R, uint32_t rid_base,
                 uint64_t seed, int64_t steps, const da_schedule &s, const LaunchShape &sh) {
    JobDesc J{};
    J.W = ctx->d_W;
    J.b = ctx->d_b;
    J.N = ctx->N;
    J.ld = ctx->ld;
    J.dtype = ctx->dtype;
    J.wscale = ctx->wscale;
    J.h = ctx->st.h;
    J.x = ctx->st.x;
    J.bx = ctx->st.bx;
    J.E = ctx->st.E;
    J.bE = ctx->st.bE;
    J.eoff = ctx->st.eoff;
    J.nacc = ctx->st.nacc;
    J.R = R;
    J.rid_base = rid_base;
    J.seed = seed;
    J.s0 = 0;
    J.s1 = steps;
    J.S = steps;
    J.L = 1;
    // increments above 2^30 act as 2^30: the offset saturates there at once
    J.eoff_inc = std::min<int32_t>(s.eoff_inc, kEoffMax);
    J.single = s.trial == DA_TRIAL_SINGLE ? 1 : 0;
    J.ell = ctx->d_ell;
    J.ell_D = ctx->ell_D;
    J.lvl_of_rep = nullptr;
    J.round_ptr = nullptr;
    J.K = 0;
    J.NW = sh.NW;
    J.NH = sh.NH;
    J.RPW = sh.RPW;
    J.w_lds = sh.w_lds;
    J.qcap = sh.qcap;
    J.ecap = sh.ecap;
    J.w24 = sh.w24;
    J.F = sh.wave ? sh.F : 0;
    J.wclamp = sh.wclamp;
    if (lt) {
        J.L = lt->L;
        J.hdr = lt->d_hdr;
        J.brk = lt->d_brk;
        J.thr = lt->d_thr;
        J.q8 = sh.direct ? lt->d_q8 : nullptr;
        J.gth = (sh.gen && lt->any_gth && s.trial != DA_TRIAL_SINGLE) ? 1 : 0;
    }
    return J;
}

bool wave_takes(int32_t dtype, int64_t hbound, int32_t wscale, double T_min, double T_max,
                LaunchShape &sh) {
    const int64_t ws = std::abs((int64_t)wscale), hb = hbound + 1;
    // the field update's factor: 16 bits for 16-bit couplings, else 24
    sh.w24 = dtype < 4 || (hbound / ws < (1 << 23) && ws < (1 << 23)) ? 1 : 0;
    const int64_t wlim = dtype == 2 ? (1 << 15) : (sh.w24 ? (1 << 23) : INT64_MAX);
    if (ws >= wlim) return false;
    // the test's sum |h| + E_off + L(u) stays below 2^31: E_off is cut off at
    // max |h| + 1, L(u) <= 11.79 T, and T 2^q < 2^17 wherever q > 0
    const double room = 2147483648.0 - 65536.0;
    if (2.0 * (double)hb + 11.8 * T_max * (1.0 + 1e-4) > room) return false;
    int q = 0;
    while (q < 17 && 2.0 * (double)(hb << (q + 1)) + 2097152.0 <= room && (ws << (q + 1)) < wlim) ++q;
    sh.qcap = q;
    // the form without a conversion needs T 2^q < 2^18; from T 2^q = 2^14 down
    // costs of zero would fall in its bracket often enough to matter (one in
    // T 2^q / 4 of them)
    sh.wclamp = T_max >= 262144.0 || T_min * (double)(1 << q) < 16384.0 ? 1 : 0;
    sh.ecap = (int)hb;
    sh.wave = true;
    return true;
}

bool wave_shape(const da_ctx *ctx, int32_t R, double T_min, double T_max, LaunchShape &sh) {
    if (ctx->ell_D > 0 || !wave_takes(ctx->dtype, ctx->hbound, ctx->wscale, T_min, T_max, sh))
        return false;
    // Up to 512 variables one wave.  Beyond, with few replicas on a compute unit,
    // a team of 8 flips per lane whose random-number waves keep the draws off the
    // step's chain; they draw two blocks a lane while that leaves them off it, one
    // where replicas share the unit, and are left out where it is full; 16 flips
    // per lane, the fewest instructions per step, where it is, or past 16 waves.
    // ns per step measured (Gaussian int16, levels of 100 steps and more) at N = 1024
    // and 1, 2, 3, 4 replicas per unit: two blocks 524, 552, 679, 725, one block 521,
    // 557, 550, 596, one wave of 16 flips 663, 680, 670, 673; N = 2048: two blocks
    // 608, 846, 1202, 1509, one block 641, 713, 887, 1333, one team of two waves of
    // 16 flips 804, 1149, 1543, 1561; N = 4096 and 1, 2, 3 per unit: 8 flips and two
    // blocks 798, 1183, 1761, 16 flips and two blocks 770, 1047, 1639, none 917,
    // 1306, 1725; N = 8192 and 1, 2: 16 flips and two blocks 1164, 2077, none 1322,
    // 2093.
    // Past three replicas per unit at N <= 1024 a call alone and calls that share
    // the chip differ: two anneals at once take what one of twice the replicas
    // takes.  Teams of one block (alone; one of two at once) against one wave at
    // 4 per unit 596; 619 against 673; 508, at 5: 730; 748 against 1000; 703 (the
    // fifth wave shares a SIMD, and the step takes as long as with eight), at 6:
    // 837; 830 against 997; 706, at 9: 1332; 1162 against 1400; 1100, from 7 on
    // otherwise slower both ways (7: 1117 against 1000).  So teams up to three, and
    // at five, where they gain 27 % alone and lose 6 % beside another.
    const int N = ctx->N;
    const int per_cu = (R + ctx->cus - 1) / ctx->cus;
    int HB = 0;   // Philox blocks per lane of a random-number wave
    if (N <= 512) {
        sh.F = N <= 64 ? 1 : N <= 128 ? 2 : N <= 256 ? 4 : 8;
    } else if (N <= 1024) {
        const bool team = per_cu <= 3 || per_cu == 5;
        sh.F = team ? 8 : 16;
        HB = !team ? 0 : per_cu <= 2 ? 2 : 1;
    } else if (N <= 2048) {
        sh.F = per_cu <= 4 ? 8 : 16;
        HB = per_cu <= 1 ? 2 : per_cu <= 4 ? 1 : 0;
    } else {
        sh.F = N <= 4096 && per_cu <= 1 ? 8 : 16;
        HB = per_cu <= (N <= 4096 ? 2 : 1) ? 2 : 0;
    }
    sh.NW = (N + 64 * sh.F - 1) / (64 * sh.F);
    sh.NH = HB > 0 ? (N + 512 * HB - 1) / (512 * HB) : 0;
    sh.direct = sh.gen = 0;
    // One wave: W in LDS where a workgroup's share of the replicas leaves it room
    // (shared by all of them), read there at a quarter of the latency
    const int64_t w_bytes = (int64_t)N * ctx->ld * ctx->dtype;
    sh.w_lds = N <= 512 && w_bytes + 32768 <= (int64_t)device_lds_limit() ? 1 : 0;
    sh.RPW = sh.NW > 1 ? 1 : sh.w_lds ? std::min(per_cu, 16) : std::min(per_cu, 4);
    sh.threads = 64 * sh.RPW * (sh.NW + sh.NH);
    sh.blocks = (R + sh.RPW - 1) / sh.RPW;
    sh.lds = wave_lds_bytes(sh.F, ctx->N, sh.NW, sh.NH, sh.RPW, sh.w_lds ? w_bytes : 0);
    return true;
}

JobDesc matrix_job(const da_ctx *ctx) {
    JobDesc J{};
    J.W = ctx->d_W;
    J.b = ctx->d_b;
    J.N = ctx->N;
    J.ld = ctx->ld;
    J.dtype = ctx->dtype;
    J.wscale = ctx->wscale;
    return J;
}

int init_state(da_ctx *ctx, const JobDesc &J, int init, hipStream_t stream) {
    int e;
    if (init == DA_INIT_ZEROS) {
        e = launch_state_zero(J, stream);
    } else {
        e = launch_rand_bits(J.x, J.R, J.N, J.ld, J.rid_base, J.seed, stream);
        const int planes = coupling_planes(ctx->dtype, ctx->hbound, ctx->wscale);
        if (!e) e = launch_fields(J, planes, J.x, J.R, J.h, stream);
        if (!e) e = launch_finish_start(J, stream);
    }
    return check_hip(ctx, (hipError_t)e, "state initialisation launch");
}

int device_lds_limit() {
    static int limit = -1;
    if (limit < 0) {
        int dev = 0;
        hipDeviceProp_t p;
        limit = 64 * 1024;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess &&
            p.sharedMemPerBlock > 0)
            limit = (int)p.sharedMemPerBlock;
    }
    return limit;
}

LaunchShape batch_shape(const da_ctx *ctx, int32_t R, const da_schedule &s) {
    LaunchShape sh;
    if (wave_shape(ctx, R, std::min(s.T_hi, s.T_lo), std::max(s.T_hi, s.T_lo), sh)) return sh;
    sh = LaunchShape();
    sh.NH = 0;
    sh.F = 8;
    sh.NW = (ctx->N + 511) / 512;
    sh.RPW = 16 / sh.NW;
    sh.w_lds = 0;
    sh.threads = 1024;
    sh.lds = run_lds_bytes(sh.NW, sh.RPW, sh.F, 0, 1, 0, ctx->ell_D > 0);
    // per-draw estimates evaluated by the compute lanes, as for anneals: fields
    // of many coupling units within the path's int32 bound, dense rows
    sh.gen = (ctx->ell_D == 0 && ctx->hbound <= kGenFieldMax &&
              ctx->hbound >= 4096 * (int64_t)std::abs(ctx->wscale))
                 ? 1
                 : 0;
    return sh;
}

int BatchRunner::prepare(std::string &err) {
    if (exec[0] && exec[1]) return DA_OK;
    int dev = 0, cus = 0;
    hipError_t qe = hipGetDevice(&dev);
    if (qe == hipSuccess) qe = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (qe != hipSuccess || cus < 1) {
        err = std::string("batch runner: device query failed: ") + hipGetErrorString(qe);
        return DA_EDEVICE;
    }
    blocks = cus;
    lds = 0;
    // room for any job, sparse row lists' delta buffers included
    for (int nw = 1; nw <= 16; ++nw)
        lds = std::max(lds, run_lds_bytes(nw, 16 / nw, 8, 0, 1, 0, true));
    if (hipMalloc(&d_jobs, sizeof(JobDesc) * kCapJobs) != hipSuccess ||
        hipMalloc(&d_items, sizeof(BatchItem) * kCapItems) != hipSuccess ||
        hipMalloc(&d_rest, sizeof(BatchItem) * kCapItems) != hipSuccess ||
        hipMalloc(&d_n, 4) != hipSuccess || hipMalloc(&d_counter, 4) != hipSuccess ||
        hipHostMalloc(&h_jobs, sizeof(JobDesc) * kCapJobs) != hipSuccess ||
        hipHostMalloc(&h_items, sizeof(BatchItem) * kCapItems) != hipSuccess ||
        hipHostMalloc(&h_rest, sizeof(BatchItem) * kCapItems) != hipSuccess ||
        hipHostMalloc(&h_n, 4) != hipSuccess) {
        err = "batch descriptor allocation failed";
        release();
        return DA_ENOMEM;
    }
    bool made = hipStreamCreateWithFlags(&cap_stream, hipStreamNonBlocking) == hipSuccess &&
                hipEventCreateWithFlags(&fork, hipEventDisableTiming) == hipSuccess;
    for (int b = 0; b < kSide && made; ++b)
        made = hipStreamCreateWithFlags(&side[b], hipStreamNonBlocking) == hipSuccess &&
               hipEventCreateWithFlags(&join[b], hipEventDisableTiming) == hipSuccess;
    if (!made) {
        err = "stream creation failed";
        release();
        return DA_EDEVICE;
    }
    // capture: counter reset (a fill kernel, no memset node) + persistent kernel
    const char *stage = "begin capture";
    hipError_t e = hipSuccess;
    for (int v = 0; v < 2 && e == hipSuccess; ++v) {
        stage = "begin capture";
        e = hipStreamBeginCapture(cap_stream, hipStreamCaptureModeThreadLocal);
        if (e == hipSuccess) {
            stage = "counter reset node";
            e = (hipError_t)launch_fill_i32(d_counter, 0, 1, cap_stream);
            if (e == hipSuccess) {
                stage = "kernel node";
                e = (hipError_t)launch_batch(d_jobs, d_rest, d_n, d_counter, blocks, 1024, lds,
                                             cap_stream, v == 1);
            }
            const hipError_t e2 = hipStreamEndCapture(cap_stream, &graph[v]);
            if (e == hipSuccess) {
                stage = "end capture";
                e = e2;
            }
        }
        if (e == hipSuccess) {
            stage = "instantiate";
            e = hipGraphInstantiate(&exec[v], graph[v], nullptr, nullptr, 0);
        }
    }
    if (e != hipSuccess) {
        err = std::string("batch graph capture failed at ") + stage + ": " + hipGetErrorString(e);
        release();
        return DA_EDEVICE;
    }
    return DA_OK;
}

namespace {
// Shape of a job among others: at most 8 waves a workgroup.  A replica's step is
// the limit (16 jobs of N = 64 .. 2048, 10^4 steps: 10.7 ms; 13.5 with 16 flips
// per lane throughout) unless the batch holds more waves than the chip does at
// once (full): then the shapes with the fewest instructions.
void mix_shape(JobDesc &J, bool full) {
    const int N = J.N;
    J.F = N <= 64 ? 1 : N <= 128 ? 2 : N <= 256 ? 4 : N <= 512 ? 8 : !full && N <= 2048 ? 8 : 16;
    J.NW = (N + 64 * J.F - 1) / (64 * J.F);
    J.NH = J.NW > 1 && !full && N <= 4096 ? (N + 1023) / 1024 : 0;
    J.RPW = J.NW > 1 ? 1 : 4;
    J.w_lds = J.F <= 2 && (int64_t)N * J.ld * J.dtype <= 32768 ? 1 : 0;
}
// A replica-step's time, roughly, in 100 ns (the order of the items only).
int mix_weight(int N) {
    int w = 2;
    for (int n = 64; n < N; n <<= 1) ++w;
    return w;
}
}  // namespace

struct BatchPlan {
    struct Mixed {
        int cls;        // coupling type and mode
        int64_t cost;
        BatchItem it;
    };
    std::vector<JobDesc> jobs;        // in their shapes
    std::vector<Mixed> mixed;         // items of the wave and team kernels, class by class
    size_t class_lds[9] = {};
    std::vector<BatchItem> rest;      // items of the batched step kernel
    bool dynamic = false;             // one of them needs its per-job features
};

int BatchRunner::run(const std::vector<JobDesc> &jobs, hipStream_t s, std::string &err) {
    int rc = prepare(err);
    if (rc) return rc;
    if (jobs.size() > (size_t)kCapJobs) {
        err = "too many jobs in one batch";
        return DA_EINVAL;
    }
    BatchPlan P;
    P.jobs = jobs;
    rc = plan_mixed(P, err);
    if (rc) return rc;
    plan_rest(P);
    note_shapes(P);
    const size_t items = std::max(P.mixed.size(), P.rest.size());
    if (items == 0) return DA_OK;
    std::memcpy(h_jobs, P.jobs.data(), P.jobs.size() * sizeof(JobDesc));
    hipError_t e = hipMemcpyAsync(d_jobs, h_jobs, P.jobs.size() * sizeof(JobDesc),
                                  hipMemcpyHostToDevice, s);
    for (size_t off = 0; off < items && e == hipSuccess; off += kCapItems) {
        // the chunk before must be done with the item tables before they change
        if (off) e = hipStreamSynchronize(s);
        if (e == hipSuccess) e = enqueue(P, off, s);
    }
    if (e != hipSuccess) {
        err = std::string("batch launch failed: ") + hipGetErrorString(e);
        settle(s);
        return DA_EDEVICE;
    }
    return DA_OK;
}

// Waits for whatever a failed batch has enqueued: the next batch rewrites the
// descriptor tables, and the caller may free the jobs' memory.
void BatchRunner::settle(hipStream_t s) {
    (void)hipStreamSynchronize(s);
    for (hipStream_t b : side) (void)hipStreamSynchronize(b);
}

int BatchRunner::plan_mixed(BatchPlan &P, std::string &err) {
    int64_t waves = 0;
    auto takes = [](const JobDesc &J) { return J.F > 0 && J.s1 > J.s0; };
    for (JobDesc &J : P.jobs) {
        if (!takes(J)) continue;
        mix_shape(J, false);
        waves += (int64_t)J.R * (J.NW + J.NH);
    }
    if (waves > 32 * (int64_t)blocks)   // more than the chip holds at once
        for (JobDesc &J : P.jobs)
            if (takes(J)) mix_shape(J, true);
    int64_t class_cost[9] = {};
    for (size_t j = 0; j < P.jobs.size(); ++j) {
        const JobDesc &J = P.jobs[j];
        if (!takes(J)) continue;
        const size_t l = wave_lds_bytes(J.F, J.N, J.NW, J.NH, J.RPW,
                                        J.w_lds ? (int64_t)J.N * J.ld * J.dtype : 0);
        const char *why = job_range_error(J);
        if (!why && (J.N > 64 * J.F * J.NW || !J.G || (!J.temps && !J.stepT) || J.NW + J.NH > 8 ||
                     (J.NH > 0 && J.N > 1024 * J.NH) || l > (size_t)device_lds_limit()))
            why = "batched job outside the kernel's shapes";
        if (why) {
            err = why;
            return DA_EINVAL;
        }
        const int mode = J.stepT || J.single ? 2 : J.wclamp ? 1 : 0;
        const int cls = (J.dtype == 1 ? 0 : J.dtype == 2 ? 1 : 2) * 3 + mode;
        P.class_lds[cls] = std::max(P.class_lds[cls], l);
        const int64_t cost = (J.s1 - J.s0) * mix_weight(J.N);
        for (int32_t r0 = 0; r0 < J.R; r0 += J.RPW)
            P.mixed.push_back(BatchPlan::Mixed{cls, cost, BatchItem{(int32_t)j, r0}});
        class_cost[cls] = std::max(class_cost[cls], cost);
    }
    // longest first within a class, and the class with the longest first
    typedef BatchPlan::Mixed Item;
    std::stable_sort(P.mixed.begin(), P.mixed.end(), [&](const Item &p, const Item &q) {
        if (p.cls != q.cls)
            return class_cost[p.cls] != class_cost[q.cls] ? class_cost[p.cls] > class_cost[q.cls]
                                                          : p.cls < q.cls;
        return p.cost > q.cost;
    });
    return DA_OK;
}

void BatchRunner::plan_rest(BatchPlan &P) {
    for (size_t j = 0; j < P.jobs.size(); ++j) {
        const JobDesc &J = P.jobs[j];
        if (J.F > 0 || J.s1 <= J.s0) continue;
        P.dynamic = P.dynamic || J.single || J.stepT || J.ell;
        for (int32_t r0 = 0; r0 < J.R; r0 += J.RPW) P.rest.push_back(BatchItem{(int32_t)j, r0});
    }
    // longest items first so the tail of the persistent launch is short
    std::stable_sort(P.rest.begin(), P.rest.end(), [&](const BatchItem &p, const BatchItem &q) {
        const JobDesc &a = P.jobs[(size_t)p.job], &b = P.jobs[(size_t)q.job];
        return (a.s1 - a.s0) * a.NW > (b.s1 - b.s0) * b.NW;
    });
}

// What each job runs in, as da_last_kernel_stats reports it: its class's launch of
// 512 threads a workgroup, or the persistent launch.
void BatchRunner::note_shapes(const BatchPlan &P) {
    int class_blocks[9] = {};
    for (const BatchPlan::Mixed &m : P.mixed) ++class_blocks[m.cls];
    std::vector<int> cls(P.jobs.size(), -1);
    for (const BatchPlan::Mixed &m : P.mixed) cls[(size_t)m.it.job] = m.cls;
    shapes.assign(P.jobs.size(), LaunchShape());
    for (size_t j = 0; j < P.jobs.size(); ++j) {
        const JobDesc &J = P.jobs[j];
        LaunchShape &sh = shapes[j];
        sh.wave = J.F > 0;
        sh.F = sh.wave ? J.F : 8;
        sh.NW = J.NW;
        sh.NH = J.NH;
        sh.RPW = J.RPW;
        sh.w_lds = J.w_lds;
        sh.gen = sh.wave || (J.gth && !P.dynamic) ? 1 : 0;
        sh.threads = sh.wave ? 512 : 1024;
        sh.blocks = J.s1 <= J.s0 ? 0 : sh.wave ? class_blocks[cls[j]] : blocks;
    }
}

// Items off .. off + kCapItems of both tables: the persistent launch (its idle
// workgroups end at once) and one launch per class, the first of them on s, the
// others beside it, joined to s.
hipError_t BatchRunner::enqueue(const BatchPlan &P, size_t off, hipStream_t s) {
    auto in_chunk = [&](size_t n) { return n > off ? std::min(n - off, (size_t)kCapItems) : 0; };
    const size_t nm = in_chunk(P.mixed.size()), nr = in_chunk(P.rest.size());
    for (size_t q = 0; q < nm; ++q) h_items[q] = P.mixed[off + q].it;
    for (size_t q = 0; q < nr; ++q) h_rest[q] = P.rest[off + q];
    *h_n = (int32_t)nr;
    hipError_t e = hipSuccess;
    if (nm) e = hipMemcpyAsync(d_items, h_items, nm * sizeof(BatchItem), hipMemcpyHostToDevice, s);
    if (nr && e == hipSuccess)
        e = hipMemcpyAsync(d_rest, h_rest, nr * sizeof(BatchItem), hipMemcpyHostToDevice, s);
    if (nr && e == hipSuccess) e = hipMemcpyAsync(d_n, h_n, 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipEventRecord(fork, s);
    int k = 0;   // launches so far
    if (nr && e == hipSuccess) {
        e = hipGraphLaunch(exec[P.dynamic ? 1 : 0], s);
        ++k;
    }
    for (size_t q = 0; q < nm && e == hipSuccess; ++k) {
        const int cls = P.mixed[off + q].cls;
        size_t end = q;
        while (end < nm && P.mixed[off + end].cls == cls) ++end;
        const int b = k == 0 ? -1 : (k - 1) % kSide;
        const hipStream_t st = b < 0 ? s : side[b];
        if (b >= 0) e = hipStreamWaitEvent(st, fork, 0);
        if (e == hipSuccess)
            e = (hipError_t)launch_mix(d_jobs, d_items + q, cls / 3 == 0 ? 1 : cls / 3 == 1 ? 2 : 4,
                                       cls % 3, (int)(end - q), P.class_lds[cls], st);
        q = end;
    }
    for (int b = 0; b < std::min(k - 1, kSide) && e == hipSuccess; ++b) {
        e = hipEventRecord(join[b], side[b]);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, join[b], 0);
    }
    return e;
}

void BatchRunner::release() {
    for (int v = 0; v < 2; ++v) {
        if (exec[v]) (void)hipGraphExecDestroy(exec[v]);
        if (graph[v]) (void)hipGraphDestroy(graph[v]);
        exec[v] = nullptr;
        graph[v] = nullptr;
    }
    if (cap_stream) (void)hipStreamDestroy(cap_stream);
    if (fork) (void)hipEventDestroy(fork);
    fork = nullptr;
    for (int b = 0; b < kSide; ++b) {
        if (side[b]) (void)hipStreamDestroy(side[b]);
        if (join[b]) (void)hipEventDestroy(join[b]);
        side[b] = nullptr;
        join[b] = nullptr;
    }
    for (void *p : {(void *)d_jobs, (void *)d_items, (void *)d_rest, (void *)d_n, (void *)d_counter})
        if (p) (void)hipFree(p);
    for (void *p : {(void *)h_jobs, (void *)h_items, (void *)h_rest, (void *)h_n})
        if (p) (void)hipHostFree(p);
    cap_stream = nullptr;
    d_jobs = nullptr;
    d_items = d_rest = nullptr;
    d_n = d_counter = nullptr;
    h_jobs = nullptr;
    h_items = h_rest = nullptr;
    h_n = nullptr;
}

namespace {
// Calls f(i, j, w_ij) for every pair i < j, w_ij = Q_ij + Q_ji, in 64 x 64
// tiles so that the transposed reads stay in cache.
template <class Fn>
void for_upper_pairs(const int32_t *Q, size_t n, Fn &&f) {
    constexpr size_t B = 64;
    for (size_t I = 0; I < n; I += B)
        for (size_t J = I; J < n; J += B) {
            const size_t ie = std::min(I + B, n), je = std::min(J + B, n);
            for (size_t i = I; i < ie; ++i)
                for (size_t j = std::max(J, i + 1); j < je; ++j)
                    f(i, j, (int64_t)Q[i * n + j] + (int64_t)Q[j * n + i]);
        }
}
}  // namespace

int derive_storage(const int32_t *Q, int32_t N, int32_t dtype_hint, int32_t &dtype,
                   int32_t &wscale, std::string &err) {
    const size_t n = (size_t)N;
    int64_t g = 0, maxw = 0;
    std::vector<int64_t> row(n);
    for (size_t i = 0; i < n; ++i) {
        const int64_t bi = Q[i * n + i];
        row[i] = bi < 0 ? -bi : bi;
    }
    for_upper_pairs(Q, n, [&](size_t i, size_t j, int64_t w) {
        const int64_t aw = w < 0 ? -w : w;
        row[i] += aw;
        row[j] += aw;
        maxw = std::max(maxw, aw);
        if (w && g != 1) g = gcd64(g, w);
    });
    const int64_t maxrow = n ? *std::max_element(row.begin(), row.end()) : 0;
    return choose_storage(maxrow, maxw, g, dtype_hint, dtype, wscale, err);
}

int choose_storage(int64_t maxrow, int64_t maxw, int64_t g, int32_t dtype_hint, int32_t &dtype,
                   int32_t &wscale, std::string &err) {
    if (maxrow > (int64_t(1) << 30)) {
        err = "max_i |b_i| + sum_j |W_ij| exceeds 2^30: fields would not fit int32";
        return DA_ERANGE;
    }
    if (g == 0) g = 1;
    maxw /= g;
    int dt = dtype_hint;
    if (dt == DA_DTYPE_AUTO) dt = maxw <= 127 ? 1 : (maxw <= 32767 ? 2 : 4);
    const int64_t lim = dt == 1 ? 127 : (dt == 2 ? 32767 : 2147483647);
    if (maxw > lim) {
        err = "couplings do not fit the requested type";
        return DA_ERANGE;
    }
    dtype = dt;
    wscale = (int32_t)g;
    return DA_OK;
}

namespace {
template <typename T>
void fill_padded(const int32_t *Q, size_t n, size_t ld, int64_t g, uint8_t *dst,
                 std::vector<int64_t> &row) {
    T *W = reinterpret_cast<T *>(dst);
    for_upper_pairs(Q, n, [&](size_t i, size_t j, int64_t w) {
        const T v = (T)(w / g);
        W[i * ld + j] = v;
        W[j * ld + i] = v;
        const int64_t aw = w < 0 ? -w : w;
        row[i] += aw;
        row[j] += aw;
    });
}
}  // namespace

void prepare_matrix(const int32_t *Q, int32_t N, int32_t dtype, int32_t wscale, HostMatrix &hm) {
    hm.N = N;
    hm.ld = (N + 63) / 64 * 64;
    hm.dtype = dtype;
    hm.wscale = wscale;
    const size_t n = (size_t)N, ld = (size_t)hm.ld;
    hm.W.assign(ld * ld * (size_t)dtype, 0);
    std::vector<int64_t> row(n, 0);
    if (dtype == 1) fill_padded<int8_t>(Q, n, ld, wscale, hm.W.data(), row);
    else if (dtype == 2) fill_padded<int16_t>(Q, n, ld, wscale, hm.W.data(), row);
    else fill_padded<int32_t>(Q, n, ld, wscale, hm.W.data(), row);
    hm.b.assign(ld, 0);
    hm.hbound = 0;
    for (size_t i = 0; i < n; ++i) {
        hm.b[i] = Q[i * n + i];
        hm.hbound = std::max(hm.hbound, row[i] + (hm.b[i] < 0 ? -(int64_t)hm.b[i] : hm.b[i]));
    }
}

int prepare_sparse(const int32_t *Q, int32_t N, HostMatrix &hm, std::string &err) {
    const size_t n = (size_t)N;
    const int64_t g = hm.wscale;
    std::vector<std::vector<uint32_t>> rows(n);
    for (size_t i = 0; i < n; ++i)
        for (size_t j = 0; j < n; ++j) {
            if (i == j) continue;
            const int64_t w = ((int64_t)Q[i * n + j] + (int64_t)Q[j * n + i]) / g;
            if (!w) continue;
            if (w < -32768 || w > 32767) {
                err = "a coupling does not fit the 16-bit sparse entry";
                return DA_ERANGE;
            }
            rows[i].push_back((uint32_t)j | ((uint32_t)(uint16_t)(int16_t)w << 16));
        }
    size_t D = 4;
    for (auto &r : rows) D = std::max(D, (r.size() + 3) / 4 * 4);
    if (D > 1024) {
        err = "a row has more than 1024 nonzeros: use dense storage";
        return DA_ERANGE;
    }
    hm.ell_D = (int32_t)D;
    hm.ell.assign(n * D, 0xFFFFu);   // padding: column 0xFFFF, value 0
    for (size_t i = 0; i < n; ++i)
        std::copy(rows[i].begin(), rows[i].end(), hm.ell.begin() + (ptrdiff_t)(i * D));
    return DA_OK;
}

int create_ctx(const HostMatrix &hm, hipStream_t s, da_ctx **out, std::string &err,
               const int32_t *d_Q) {
    da_ctx *ctx = new (std::nothrow) da_ctx();
    if (!ctx) {
        err = "host allocation failed";
        return DA_ENOMEM;
    }
    ctx->N = hm.N;
    ctx->ld = hm.ld;
    ctx->dtype = hm.dtype;
    ctx->wscale = hm.wscale;
    ctx->hbound = hm.hbound;
    const char *what = nullptr;
    hipError_t e = hipGetDevice(&ctx->device);
    if (e != hipSuccess) what = "device query";
    if (!what && (e = hipDeviceGetAttribute(&ctx->cus, hipDeviceAttributeMultiprocessorCount,
                                            ctx->device)) != hipSuccess)
        what = "compute-unit count";
    const size_t w_bytes = (size_t)hm.ld * hm.ld * (size_t)hm.dtype;
    if (!what && (e = hipMalloc(&ctx->d_W, w_bytes)) != hipSuccess) what = "W allocation";
    if (!what && (e = hipMalloc(&ctx->d_b, (size_t)hm.ld * 4)) != hipSuccess) what = "b allocation";
    if (!what && d_Q &&
        (e = (hipError_t)launch_image(d_Q, hm.N, hm.ld, hm.dtype, hm.wscale, ctx->d_W, ctx->d_b, s)) !=
            hipSuccess)
        what = "instance image";
    if (!what && !d_Q && (e = hipMemcpyAsync(ctx->d_W, hm.W.data(), hm.W.size(), hipMemcpyHostToDevice,
                                     s)) != hipSuccess)
        what = "W upload";
    if (!what && !d_Q && (e = hipMemcpyAsync(ctx->d_b, hm.b.data(), hm.b.size() * 4,
                                     hipMemcpyHostToDevice, s)) != hipSuccess)
        what = "b upload";
    if (!what && hm.ell_D > 0) {
        ctx->ell_D = hm.ell_D;
        if ((e = hipMalloc(&ctx->d_ell, hm.ell.size() * 4)) != hipSuccess) what = "sparse allocation";
        else if ((e = hipMemcpyAsync(ctx->d_ell, hm.ell.data(), hm.ell.size() * 4,
                                     hipMemcpyHostToDevice, s)) != hipSuccess)
            what = "sparse upload";
    }
    // the host image may be freed when this returns
    if (!what && (e = hipStreamSynchronize(s)) != hipSuccess) what = "upload";
    if (!what && (e = hipStreamCreateWithFlags(&ctx->own_stream, hipStreamNonBlocking)) !=
                     hipSuccess)
        what = "stream";
    if (what) {
        err = std::string(what) + ": " + hipGetErrorString(e);
        da_destroy(ctx);
        return (e == hipErrorOutOfMemory) ? DA_ENOMEM : DA_EDEVICE;
    }
    *out = ctx;
    return DA_OK;
}

TempList::~TempList() {
    if (d_temps) (void)hipFree(d_temps);
}

namespace {
std::mutex g_temps_mu;
std::map<std::string, std::weak_ptr<TempList>> g_temps;
std::mutex g_gerr_mu;
std::map<int, float> g_gerr;
}  // namespace

std::shared_ptr<TempList> get_temp_list(const std::vector<double> &temps, std::string &err) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        err = "hipGetDevice failed";
        return nullptr;
    }
    std::string key(reinterpret_cast<const char *>(&dev), sizeof dev);
    key.append(reinterpret_cast<const char *>(temps.data()), temps.size() * sizeof(double));
    std::lock_guard<std::mutex> lock(g_temps_mu);
    auto it = g_temps.find(key);
    if (it != g_temps.end()) {
        if (auto sp = it->second.lock()) return sp;
    }
    auto tl = std::make_shared<TempList>();
    const size_t bytes = temps.size() * sizeof(double);
    // (T = 0 schedules give 0 x NaN past their first level)
    std::vector<double> pos(temps);
    for (double &T : pos) T = T > 0.0 ? T : 0.0;
    if (hipMalloc(&tl->d_temps, bytes) != hipSuccess ||
        hipMemcpy(tl->d_temps, pos.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) {
        err = "temperature list allocation or upload failed";
        return nullptr;
    }
    // (lists that no context holds any more leave the cache here)
    for (auto q = g_temps.begin(); q != g_temps.end();)
        q = q->second.expired() ? g_temps.erase(q) : std::next(q);
    g_temps[key] = tl;
    return tl;
}

// The error of tt(u) of the one-wave kernel per unit of T 2^q (da_wave.hip):
// the fp32 roundings of its three terms, (16 + 16 + 17) ln 2 2^-24 = 2.03e-6,
// and ln 2 times the device's log2 error, which is measured.
bool device_bound_error(float &gerr, std::string &err) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        err = "hipGetDevice failed";
        return false;
    }
    const double *G = device_neg_log_u(err);
    if (!G) return false;
    std::lock_guard<std::mutex> lock(g_gerr_mu);
    auto it = g_gerr.find(dev);
    if (it == g_gerr.end()) {
        float *d = nullptr, e = 0.0f;
        const bool ok = hipMalloc(&d, sizeof *d) == hipSuccess &&
                        launch_log_error(G, d, nullptr) == hipSuccess &&
                        hipMemcpy(&e, d, sizeof e, hipMemcpyDeviceToHost) == hipSuccess;
        if (d) (void)hipFree(d);
        if (!ok) {
            err = "log2 error pass failed";
            return false;
        }
        it = g_gerr.emplace(dev, 0.6932f * e + 2.2e-6f).first;
    }
    gerr = it->second;
    return true;
}

// ---------------------------------------------------------------------------
// Autotuner.  Launch shapes never change results, only speed, so the first
// anneal of each (device, N, coupling type, replica-count bucket) times every
// candidate shape on a window of its own schedule, run on scratch state, and
// keeps the fastest for later calls.  DAPT_AUTOTUNE=0 disables it.
// ---------------------------------------------------------------------------
namespace {
struct TuneKey {
    int dev, N, dtype, rbucket;
    int direct;
    bool operator<(const TuneKey &o) const {
        if (dev != o.dev) return dev < o.dev;
        if (N != o.N) return N < o.N;
        if (dtype != o.dtype) return dtype < o.dtype;
        if (rbucket != o.rbucket) return rbucket < o.rbucket;
        return direct < o.direct;
    }
};
std::mutex g_tune_mu;
std::map<TuneKey, da_launch> g_tune;

bool tune_enabled() {
    const char *e = std::getenv("DAPT_AUTOTUNE");
    return !(e && e[0] == '0');
}
}  // namespace

// Direct tables pay for their staging (64 KiB per level and workgroup) only
// when levels last a few hundred steps.
static bool want_direct(const LevelTables &lt, const da_schedule &sched, int64_t steps) {
    return lt.d_q8 != nullptr && sched.n_levels > 0 && steps >= 256 * (int64_t)sched.n_levels;
}

int tuned_shape(da_ctx *ctx, const LevelTables &lt, int32_t R, int64_t steps,
                const da_schedule &sched, hipStream_t s, bool may_time, LaunchShape &out) {
    const bool direct = want_direct(lt, sched, steps);
    int rc = DA_OK, rb = 1;
    while (rb < R) rb <<= 1;
    // (long levels have direct tables, and other shapes win there)
    const TuneKey key{ctx->device, ctx->N, ctx->dtype, rb, direct ? 1 : 0};
    {
        std::lock_guard<std::mutex> lock(g_tune_mu);
        auto it = g_tune.find(key);
        if (it != g_tune.end()) {
            out = choose_shape(ctx, R, &it->second, true, direct);
            return DA_OK;
        }
    }
    const int64_t window = std::min<int64_t>(steps, 384);
    out = choose_shape(ctx, R, nullptr, true, direct);
    if (window < 64 || !may_time) return DA_OK;
    // The candidates run on the context's own replica state (it must hold R
    // replicas already); the caller initialises it for the real run afterwards.
    if (ctx->st.cap < R || ctx->st.ld != ctx->ld)
        return fail(ctx, DA_EINVAL, "autotuner: replica state not allocated");
    hipEvent_t a = nullptr, b = nullptr;
    rc = check_hip(ctx, hipEventCreate(&a), "autotuner: event create");
    if (!rc) rc = check_hip(ctx, hipEventCreate(&b), "autotuner: event create");
    da_launch best{0, 0, 0, 0, 0};
    float best_ms = 1e30f;
    auto time_candidate = [&](JobDesc J, const LaunchShape &sh, const da_launch &cand,
                              const char *what) {
        tune_window(steps, J.s0, J.s1);
        if (const char *why = job_range_error(J)) {
            rc = fail(ctx, DA_EINVAL, std::string("autotuner: ") + why);
            return;
        }
        rc = check_hip(ctx, (hipError_t)launch_state_zero(J, s), what);
        if (!rc) rc = check_hip(ctx, hipEventRecord(a, s), what);
        if (!rc)
            rc = check_hip(ctx,
                           (hipError_t)launch_run(J, sh.F, sh.NH > 0, nullptr, sh.blocks,
                                                  sh.threads, sh.lds, s),
                           what);
        if (!rc) rc = check_hip(ctx, hipEventRecord(b, s), what);
        if (!rc) rc = check_hip(ctx, hipEventSynchronize(b), what);
        float ms = 0.f;
        if (!rc) rc = check_hip(ctx, hipEventElapsedTime(&ms, a, b), what);
        if (!rc && ms < best_ms) {
            best_ms = ms;
            best = cand;
        }
    };
    // W staged in LDS is a candidate whenever it fits there
    const bool w_fits = ctx->ell_D == 0 &&
                        (int64_t)ctx->N * ctx->ld * ctx->dtype <= (int64_t)device_lds_limit();
    for (int F : {2, 4, 8}) {
        if (F == 2 && ctx->dtype > 2) continue;
        for (int rpw : {1, 2, 4}) {
            for (int rng : {1, -1})
            for (int wl : {-1, 1})
            for (int ge : {1, -1}) {
                if (rc) break;
                if (wl > 0 && !w_fits) continue;
                const da_launch cand{F, rpw, wl, rng, ge};
                const LaunchShape sh = choose_shape(ctx, R, &cand, true, direct);
                if (sh.RPW != rpw || sh.F != F || sh.w_lds != (wl > 0 ? 1 : 0) ||
                    sh.threads > 1024 || sh.lds > (size_t)device_lds_limit())
                    continue;
                // the estimate candidate only where the shape can take it
                if (ge > 0 && (!sh.gen || !lt.any_gth)) continue;
                JobDesc J = make_job(ctx, &lt, R, 0u, 1u, steps, sched, sh);
                // any failure here is a device fault or a launch the device
                // refused: report it with the candidate instead of moving on
                char what[160];
                std::snprintf(what, sizeof what,
                              "autotuner candidate (flips/lane %d, replicas/workgroup %d, "
                              "rng waves %d, W in LDS %d, draw estimates %d)", F, rpw, rng, wl,
                              ge);
                time_candidate(J, sh, cand, what);
            }
        }
    }
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
    if (rc) return rc;
    if (best.flips_per_lane == 0) return DA_OK;
    {
        std::lock_guard<std::mutex> lock(g_tune_mu);
        g_tune[key] = best;
    }
    out = choose_shape(ctx, R, &best, true, direct);
    return DA_OK;
}

int next_events(da_ctx *ctx, hipEvent_t &e0, hipEvent_t &e1) {
    if (ctx->ev_used == kEventPool) {
        // fold the window into running totals so the pool stays bounded
        int rc = check_hip(ctx, hipEventSynchronize(ctx->ev1), "event synchronise");
        for (size_t q = 0; q < ctx->ev_used && !rc; ++q) {
            float ms = 0.f;
            rc = check_hip(ctx, hipEventElapsedTime(&ms, ctx->ev_pool[q].first, ctx->ev_pool[q].second),
                           "event elapsed time");
            ctx->folded_ms += ms;
        }
        if (rc) return rc;
        ctx->folded_calls += (int64_t)ctx->ev_used;
        ctx->ev_used = 0;
    }
    if (ctx->ev_used == ctx->ev_pool.size()) {
        hipEvent_t a = nullptr, b = nullptr;
        int rc = check_hip(ctx, hipEventCreate(&a), "event create");
        if (!rc) rc = check_hip(ctx, hipEventCreate(&b), "event create");
        if (rc) return rc;
        ctx->ev_pool.emplace_back(a, b);
    }
    e0 = ctx->ev_pool[ctx->ev_used].first;
    e1 = ctx->ev_pool[ctx->ev_used].second;
    ++ctx->ev_used;
    ctx->ev0 = e0;
    ctx->ev1 = e1;
    return DA_OK;
}

int job_tables(const da_schedule &sch, int64_t steps, bool wave, JobTables &jt, std::string &err,
               const HostTables *pre) {
    if (sch.n_levels == 0 && steps > kMaxPerStepSteps) {
        err = "per-step schedules take at most 2^24 steps";
        return DA_EINVAL;
    }
    const bool perstep = sch.n_levels == 0 && steps > 0;
    if (perstep) {
        jt.steps = get_step_tables(sch, steps, err);
        if (!jt.steps) return DA_ENOMEM;
    }
    if (wave) {
        if (!perstep) {
            jt.temps = get_temp_list(
                sch.n_levels > 0 ? schedule_temps(sch) : std::vector<double>{0.0}, err);
            if (!jt.temps) return DA_ENOMEM;
        }
        if (!device_bound_error(jt.gerr, err)) return DA_ENOMEM;
    } else {
        jt.levels = get_level_tables(
            sch.n_levels > 0 ? schedule_temps(sch) : std::vector<double>{0.0}, err, pre);
        if (!jt.levels) return DA_ENOMEM;
    }
    if (wave || perstep) {
        jt.G = device_neg_log_u(err);
        if (!jt.G) return DA_ENOMEM;
    }
    return DA_OK;
}

void attach_tables(JobDesc &J, const da_schedule &sch, const JobTables &jt) {
    J.stepT = jt.steps ? jt.steps->d_steps : nullptr;
    J.G = jt.G;
    J.temps = jt.temps ? jt.temps->d_temps : nullptr;
    J.gerr = jt.gerr;
    if (jt.temps) J.L = std::max(sch.n_levels, 1);
}

namespace {
// Pinned blocks that small outputs pass through: at most kBlocks per process,
// allocated when first needed, each with one call at a time, kept until the
// process ends.  A call that finds none free copies to the caller's memory.
class PinnedBlocks {
  public:
    static constexpr size_t kBytes = size_t(1) << 20;
    static constexpr int kBlocks = 8;
    void *take() {
        std::lock_guard<std::mutex> lock(mu_);
        if (!free_.empty()) {
            void *p = free_.back();
            free_.pop_back();
            return p;
        }
        void *p = nullptr;
        if (made_ == kBlocks) return nullptr;
        if (hipHostMalloc(&p, kBytes, hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();   // (or the next launch reports it)
            return nullptr;
        }
        ++made_;
        return p;
    }
    void give(void *p) {
        std::lock_guard<std::mutex> lock(mu_);
        free_.push_back(p);
    }

  private:
    std::mutex mu_;
    std::vector<void *> free_;
    int made_ = 0;
};
PinnedBlocks &pinned_blocks() {
    static PinnedBlocks *p = new PinnedBlocks();   // (no frees at exit)
    return *p;
}

}  // namespace

// Outputs to the caller's memory.  A kernel writes them densely, up to 1 MiB
// into a pinned block itself (one launch and one wait), more into device memory
// that contiguous copies leave from: strided copies to pageable memory go row by
// row (2048 rows of 1024 bytes took 26 ms).  That device memory is `scratch`, where
// the caller has enough to spare, or allocated in stream order for this call; where
// there is none, the rows are copied one by one.
int copy_outputs_to_host(da_ctx *ctx, const JobDesc &J, int32_t R, const da_result *o,
                         hipStream_t s, void *scratch, size_t scratch_bytes) {
    const size_t nE = (size_t)R * 8, nx = (size_t)R * (size_t)J.N;
    const size_t bytes = 3 * nE + 2 * nx;
    JobDesc K = J;
    K.R = R;
    auto parts = [&](void *at) {   // [3][R] energies and counts, then [2][R][N] states
        char *p = static_cast<char *>(at);
        da_result d{};
        d.best_E = o->best_E ? reinterpret_cast<int64_t *>(p) : nullptr;
        d.final_E = o->final_E ? reinterpret_cast<int64_t *>(p + nE) : nullptr;
        d.n_accept = o->n_accept ? reinterpret_cast<int64_t *>(p + 2 * nE) : nullptr;
        d.best_x = o->best_x ? reinterpret_cast<uint8_t *>(p + 3 * nE) : nullptr;
        d.final_x = o->final_x ? reinterpret_cast<uint8_t *>(p + 3 * nE + nx) : nullptr;
        return d;
    };
    void *pin = bytes <= PinnedBlocks::kBytes ? pinned_blocks().take() : nullptr;
    void *at = pin ? pin : bytes <= scratch_bytes ? scratch : nullptr, *own = nullptr;
    if (!at) {
        if (hipMallocAsync(&own, bytes, s) == hipSuccess) at = own;
        else (void)hipGetLastError();   // (or the next launch reports it)
    }
    hipError_t e = hipSuccess;
    if (!at) {
        auto rows = [&](uint8_t *dst, const uint8_t *src) {
            if (dst && e == hipSuccess)
                e = hipMemcpy2DAsync(dst, (size_t)J.N, src, (size_t)J.ld, (size_t)J.N, (size_t)R,
                                     hipMemcpyDeviceToHost, s);
        };
        auto words = [&](int64_t *dst, const int64_t *src) {
            if (dst && e == hipSuccess) e = hipMemcpyAsync(dst, src, nE, hipMemcpyDeviceToHost, s);
        };
        rows(o->best_x, J.bx);
        rows(o->final_x, J.x);
        words(o->best_E, J.bE);
        words(o->final_E, J.E);
        words(o->n_accept, J.nacc);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        return check_hip(ctx, e, "copy of outputs to host");
    }
    const da_result d = parts(at);
    e = (hipError_t)launch_outputs(K, d, s);
    if (pin && e == hipSuccess) e = hipStreamSynchronize(s);
    auto copy = [&](void *dst, const void *src, size_t n) {
        if (!dst || e != hipSuccess) return;
        if (pin) std::memcpy(dst, src, n);
        else e = hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToHost, s);
    };
    copy(o->best_E, d.best_E, nE);
    copy(o->final_E, d.final_E, nE);
    copy(o->n_accept, d.n_accept, nE);
    copy(o->best_x, d.best_x, nx);
    copy(o->final_x, d.final_x, nx);
    if (own) (void)hipFreeAsync(own, s);
    // (after a failed wait the kernel may still write to the block: left out of use)
    if (pin && e == hipSuccess) pinned_blocks().give(pin);
    if (!pin && e == hipSuccess) e = hipStreamSynchronize(s);
    return check_hip(ctx, e, "copy of outputs to host");
}

}  // namespace dapt

namespace {

constexpr int64_t kMaxSteps = (int64_t(1) << 31) - 1;

bool device_is_gfx950(std::string &err) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        err = std::string("no HIP device: ") + hipGetErrorString(e);
        return false;
    }
    // (a device's properties do not change; the query takes longer than a launch)
    static std::mutex mu;
    static std::map<int, std::string> arch;
    std::lock_guard<std::mutex> lock(mu);
    auto it = arch.find(dev);
    if (it == arch.end()) {
        hipDeviceProp_t p;
        e = hipGetDeviceProperties(&p, dev);
        if (e != hipSuccess) {
            err = std::string("hipGetDeviceProperties failed: ") + hipGetErrorString(e);
            return false;
        }
        it = arch.emplace(dev, p.gcnArchName).first;
    }
    if (it->second.compare(0, 6, "gfx950") != 0) {
        err = "device is " + it->second + ", this library is built for gfx950";
        return false;
    }
    return true;
}

hipStream_t ctx_stream(da_ctx *ctx, void *stream) {
    return stream ? reinterpret_cast<hipStream_t>(stream) : ctx->own_stream;
}

// Copy-out of one anneal's outputs from the context state into device buffers.
int extract_outputs(da_ctx *ctx, const JobDesc &J, int32_t R, const da_result *o, hipStream_t s) {
    JobDesc K = J;
    K.R = R;
    return check_hip(ctx, (hipError_t)launch_outputs(K, *o, s), "output extraction launch");
}

void record_stats(da_ctx *ctx, const LaunchShape &sh, int64_t launches, int gth = 0) {
    (void)launches;
    ctx->last = da_kernel_stats{};
    ctx->last.blocks = sh.blocks;
    ctx->last.threads = sh.threads;
    ctx->last.flips_per_lane = sh.F;
    ctx->last.replicas_per_block = sh.RPW;
    ctx->last.w_in_lds = sh.w_lds;
    ctx->last.rng_waves = sh.NH;
    ctx->last.dtype = ctx->dtype;
    ctx->last.draw_estimates = gth;
    ctx->have_stats = true;
}

// Enqueue a full anneal: state init, step kernel between timing events.
// Steps [step_begin, step_end) of a `steps`-step anneal; step_begin > 0
// continues from the state the context holds.
int enqueue_anneal(da_ctx *ctx, const da_schedule *schedule, int64_t replica_base,
                   int32_t replicas, int64_t steps, uint64_t seed, const da_launch *launch,
                   const da_trace *trace_dev, hipStream_t s, JobDesc &J,
                   int64_t step_begin = 0, int64_t step_end = -1) {
    std::string err;
    if (!ctx) return fail(nullptr, DA_EINVAL, "ctx is null");
    int rc = validate_schedule(schedule, err);
    if (rc) return fail(ctx, rc, err);
    if (replicas < 1) return fail(ctx, DA_EINVAL, "replicas must be >= 1");
    if (steps < 0 || steps > kMaxSteps) return fail(ctx, DA_EINVAL, "steps must be in [0, 2^31)");
    if (step_end < 0) step_end = steps;
    if (step_begin < 0 || step_begin > step_end || step_end > steps)
        return fail(ctx, DA_EINVAL, "need 0 <= step_begin <= step_end <= total steps");
    if (replica_base < 0 || replica_base + replicas > (int64_t(1) << 31))
        return fail(ctx, DA_EINVAL, "replica ids must lie in [0, 2^31)");
    if (step_begin > 0 && (ctx->st_step != step_begin || ctx->st_base != replica_base ||
                           ctx->st_R < replicas))
        return fail(ctx, DA_EINVAL, "the context holds no state of these replicas at step_begin");
    JobTables jt;
    LaunchShape sh;
    const bool own = launch == nullptr && trace_dev == nullptr;
    const bool wave = own && wave_shape(ctx, replicas, std::min(schedule->T_hi, schedule->T_lo),
                                        std::max(schedule->T_hi, schedule->T_lo), sh);
    rc = job_tables(*schedule, steps, wave, jt, err);
    if (rc) return fail(ctx, rc, err);
    ctx->keep_tables = jt.levels;
    ctx->keep_steps = jt.steps;
    ctx->keep_temps = jt.temps;
    if (!ctx->st.ensure(replicas, ctx->ld, err)) return fail(ctx, DA_ENOMEM, err);
    // from here on the state changes: it is resumable again only on success
    ctx->st_step = -1;
    // the tuner times its candidates on the replica state, so only when the
    // run starts from the initial state (which is written after it); a resumed
    // piece takes the cached choice or the default
    if (!wave) {
        if (own && tune_enabled() && schedule->n_levels > 0) {
            rc = tuned_shape(ctx, *jt.levels, replicas, steps, *schedule, s, step_begin == 0, sh);
            if (rc) return rc;
        } else {
            sh = choose_shape(ctx, replicas, launch, true,
                              !jt.steps && want_direct(*jt.levels, *schedule, steps));
        }
    }
    J = make_job(ctx, jt.levels.get(), replicas, (uint32_t)replica_base, seed, steps, *schedule, sh);
    attach_tables(J, *schedule, jt);
    J.s0 = step_begin;
    J.s1 = step_end;
    if (const char *why = job_range_error(J)) return fail(ctx, DA_EINVAL, why);
    if (step_begin == 0) {
        rc = init_state(ctx, J, schedule->init, s);
        if (rc) return rc;
    }
    hipEvent_t e0, e1;
    rc = next_events(ctx, e0, e1);
    if (rc) return rc;
    rc = check_hip(ctx, hipEventRecord(e0, s), "event record");
    if (rc) return rc;
    if (step_end > step_begin) {
        TraceDesc T{nullptr, nullptr, nullptr, steps};
        if (trace_dev) {
            T.k = trace_dev->k;
            T.E = trace_dev->E;
            T.eoff = trace_dev->eoff;
        }
        const int e = wave ? launch_wave(J, sh.F, sh.blocks, sh.threads, sh.lds, s)
                           : launch_run(J, sh.F, sh.NH > 0, trace_dev ? &T : nullptr, sh.blocks,
                                        sh.threads, sh.lds, s);
        rc = check_hip(ctx, (hipError_t)e, "step kernel launch");
        if (rc) return rc;
    }
    rc = check_hip(ctx, hipEventRecord(e1, s), "event record");
    if (rc) return rc;
    record_stats(ctx, sh, 1, wave ? 1 : J.gth);
    ctx->st_step = step_end;
    ctx->st_base = replica_base;
    ctx->st_R = replicas;
    return DA_OK;
}

}  // namespace

extern "C" {

int da_create(const int32_t *Q, int32_t N, int32_t dtype_hint, da_ctx **out) {
    if (!out) return fail(nullptr, DA_EINVAL, "out is null");
    *out = nullptr;
    if (!Q) return fail(nullptr, DA_EINVAL, "Q is null");
    if (N < 1 || N > DA_MAX_N) return fail(nullptr, DA_EINVAL, "N must be in [1, 8192]");
    const bool sparse = (dtype_hint & DA_STORE_SPARSE) != 0;
    dtype_hint &= ~DA_STORE_SPARSE;
    if (dtype_hint != DA_DTYPE_AUTO && dtype_hint != DA_DTYPE_I8 && dtype_hint != DA_DTYPE_I16 &&
        dtype_hint != DA_DTYPE_I32)
        return fail(nullptr, DA_EINVAL, "unknown dtype hint");
    std::string err;
    if (!device_is_gfx950(err)) return fail(nullptr, DA_EDEVICE, err);

    // Small instances on the host: the device's answer takes a round trip and an
    // upload buffer (us, host and device: N = 64 73 and 141, 129 102 and 178, 200 142
    // and 179, 256 236 and 186, 512 800 and 220, 8192 315 ms and 10.6)
    auto on_host = [&]() -> int {
        HostMatrix hm;
        int32_t dtype = 0, wscale = 1;
        int rc = derive_storage(Q, N, dtype_hint, dtype, wscale, err);
        if (!rc) {
            prepare_matrix(Q, N, dtype, wscale, hm);
            if (sparse) rc = prepare_sparse(Q, N, hm, err);
        }
        if (!rc) rc = create_ctx(hm, nullptr, out, err);
        return rc ? fail(nullptr, rc, err) : DA_OK;
    };
    if (N <= 224) return on_host();
    // Q and the derivation's scratch, on the device for the length of this call.
    // Ordered on the stream and given back when that is waited for: hipFree waits
    // for everything that runs on the device, other contexts' anneals too (N = 512
    // beside an anneal of 414 ms: 414 ms with it).  Where it does not fit beside the
    // image, the host derives
    const size_t q_bytes = (size_t)N * (size_t)N * 4;
    const size_t q_pad = (q_bytes + 255) & ~(size_t)255;
    char *d = nullptr;
    if (hipMallocAsync((void **)&d, q_pad + derive_scratch_bytes(N), nullptr) != hipSuccess) {
        (void)hipGetLastError();   // (or the next launch reports it)
        return on_host();
    }
    const int32_t *d_Q = reinterpret_cast<const int32_t *>(d);
    uint64_t *res = nullptr, host[3] = {0, 0, 0};
    hipError_t e = hipMemcpyAsync(d, Q, q_bytes, hipMemcpyHostToDevice, nullptr);
    if (e == hipSuccess)
        e = (hipError_t)launch_derive(d_Q, N, reinterpret_cast<uint64_t *>(d + q_pad), &res, nullptr);
    if (e == hipSuccess) e = hipMemcpyAsync(host, res, sizeof host, hipMemcpyDeviceToHost, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    int rc = check_hip(nullptr, e, "instance derivation");
    HostMatrix hm;
    hm.N = N;
    hm.ld = (N + 63) / 64 * 64;
    hm.hbound = (int64_t)host[0];
    if (!rc) {
        rc = choose_storage((int64_t)host[0], (int64_t)host[1], (int64_t)host[2], dtype_hint,
                            hm.dtype, hm.wscale, err);
        if (!rc && sparse) rc = prepare_sparse(Q, N, hm, err);
        if (!rc) rc = create_ctx(hm, nullptr, out, err, d_Q);
        if (rc) fail(nullptr, rc, err);
    }
    (void)hipFreeAsync(d, nullptr);
    (void)hipStreamSynchronize(nullptr);
    if (rc != DA_ENOMEM) return rc;
    (void)hipGetLastError();
    return on_host();
}

void da_destroy(da_ctx *ctx) {
    if (!ctx) return;
    if (ctx->own_stream) (void)hipStreamSynchronize(ctx->own_stream);
    (void)hipDeviceSynchronize();
    ctx->st.release();
    if (ctx->d_W) (void)hipFree(ctx->d_W);
    if (ctx->d_b) (void)hipFree(ctx->d_b);
    if (ctx->d_ell) (void)hipFree(ctx->d_ell);
    for (void *p : {(void *)ctx->pt_slot2rep, (void *)ctx->pt_lvl, (void *)ctx->pt_swaps,
                    (void *)ctx->pt_pair, (void *)ctx->pt_round, (void *)ctx->pt_dbeta})
        if (p) (void)hipFree(p);
    for (auto &pr : ctx->ev_pool) {
        (void)hipEventDestroy(pr.first);
        (void)hipEventDestroy(pr.second);
    }
    if (ctx->own_stream) (void)hipStreamDestroy(ctx->own_stream);
    delete ctx;
}

int da_get_info(const da_ctx *ctx, da_info *info) {
    if (!ctx || !info) return fail(nullptr, DA_EINVAL, "null argument");
    info->N = ctx->N;
    info->ld = ctx->ld;
    info->dtype = ctx->dtype;
    info->wscale = ctx->wscale;
    info->device_bytes = (int64_t)ctx->ld * ctx->ld * ctx->dtype + (int64_t)ctx->ld * 4 +
                         ctx->st.bytes() + (int64_t)ctx->N * ctx->ell_D * 4;
    info->sparse_degree = ctx->ell_D;
    info->reserved = 0;
    return DA_OK;
}

int da_anneal_async(da_ctx *ctx, const da_schedule *schedule, int64_t replica_base,
                    int32_t replicas, int64_t steps, uint64_t seed, const da_launch *launch,
                    const da_result *out_dev, void *stream) {
    if (!ctx) return fail(nullptr, DA_EINVAL, "ctx is null");
    hipStream_t s = ctx_stream(ctx, stream);
    JobDesc J;
    int rc = enqueue_anneal(ctx, schedule, replica_base, replicas, steps, seed, launch, nullptr, s, J);
    if (rc) return rc;
    if (out_dev) rc = extract_outputs(ctx, J, replicas, out_dev, s);
    return rc;
}

int da_anneal_ex(da_ctx *ctx, const da_schedule *schedule, int64_t replica_base,
                 int32_t replicas, int64_t steps, uint64_t seed, const da_launch *launch,
                 da_result *out, const da_trace *trace) {
    if (!ctx) return fail(nullptr, DA_EINVAL, "ctx is null");
    hipStream_t s = ctx->own_stream;
    da_trace dev_trace{nullptr, nullptr, nullptr};
    const size_t cells = (size_t)std::max<int64_t>(replicas, 0) * (size_t)std::max<int64_t>(steps, 0);
    int rc = DA_OK;
    if (trace && cells) {
        if (trace->k) rc = check_hip(ctx, hipMalloc(&dev_trace.k, cells * 4), "trace allocation");
        if (!rc && trace->E) rc = check_hip(ctx, hipMalloc(&dev_trace.E, cells * 8), "trace allocation");
        if (!rc && trace->eoff) rc = check_hip(ctx, hipMalloc(&dev_trace.eoff, cells * 8), "trace allocation");
        // the traced kernel writes every column it is given; give it all three
        if (!rc && !dev_trace.k) rc = check_hip(ctx, hipMalloc(&dev_trace.k, cells * 4), "trace allocation");
        if (!rc && !dev_trace.E) rc = check_hip(ctx, hipMalloc(&dev_trace.E, cells * 8), "trace allocation");
        if (!rc && !dev_trace.eoff) rc = check_hip(ctx, hipMalloc(&dev_trace.eoff, cells * 8), "trace allocation");
    }
    JobDesc J;
    if (!rc)
        rc = enqueue_anneal(ctx, schedule, replica_base, replicas, steps, seed, launch,
                            (trace && cells) ? &dev_trace : nullptr, s, J);
    if (!rc && out) rc = copy_outputs_to_host(ctx, J, replicas, out, s);
    if (!rc && trace && cells) {
        hipError_t e = hipSuccess;
        if (trace->k) e = hipMemcpy(trace->k, dev_trace.k, cells * 4, hipMemcpyDeviceToHost);
        if (e == hipSuccess && trace->E) e = hipMemcpy(trace->E, dev_trace.E, cells * 8, hipMemcpyDeviceToHost);
        if (e == hipSuccess && trace->eoff) e = hipMemcpy(trace->eoff, dev_trace.eoff, cells * 8, hipMemcpyDeviceToHost);
        rc = check_hip(ctx, e, "trace copy");
    }
    if (!rc && !out) rc = check_hip(ctx, hipStreamSynchronize(s), "stream synchronise");
    if (dev_trace.k) (void)hipFree(dev_trace.k);
    if (dev_trace.E) (void)hipFree(dev_trace.E);
    if (dev_trace.eoff) (void)hipFree(dev_trace.eoff);
    return rc;
}

int da_anneal(da_ctx *ctx, const da_schedule *schedule, int32_t replicas, int64_t steps,
              uint64_t seed, da_result *out) {
    return da_anneal_ex(ctx, schedule, 0, replicas, steps, seed, nullptr, out, nullptr);
}

int da_anneal_steps(da_ctx *ctx, const da_schedule *schedule, int64_t replica_base,
                    int32_t replicas, int64_t total_steps, int64_t step_begin,
                    int64_t step_end, uint64_t seed, da_result *out) {
    if (!ctx) return fail(nullptr, DA_EINVAL, "ctx is null");
    hipStream_t s = ctx->own_stream;
    JobDesc J;
    int rc = enqueue_anneal(ctx, schedule, replica_base, replicas, total_steps, seed, nullptr,
                            nullptr, s, J, step_begin, step_end);
    if (rc) return rc;
    if (out) return copy_outputs_to_host(ctx, J, replicas, out, s);
    return check_hip(ctx, hipStreamSynchronize(s), "stream synchronise");
}

int64_t da_state_bytes(int32_t N, int32_t replicas) {
    if (N < 1 || N > DA_MAX_N || replicas < 1) return -1;
    const int64_t n = N, r = replicas;
    return (int64_t)sizeof(da_state_header) + r * (2 * n + 4 * n) + r * (8 * 3 + 4);
}

int da_state_save(da_ctx *ctx, int32_t replicas, void *buf, size_t bytes) {
    if (!ctx || !buf) return fail(ctx, DA_EINVAL, "null argument");
    if (ctx->st_step < 0 || replicas < 1 || replicas > ctx->st_R)
        return fail(ctx, DA_EINVAL, "the context holds no anneal state for that many replicas");
    const int64_t need = da_state_bytes(ctx->N, replicas);
    if ((int64_t)bytes < need) return fail(ctx, DA_EINVAL, "buffer shorter than da_state_bytes");
    const size_t N = (size_t)ctx->N, ld = (size_t)ctx->ld, R = (size_t)replicas;
    auto *hdr = static_cast<da_state_header *>(buf);
    hdr->magic = 0x54534144u;
    hdr->version = 1;
    hdr->N = ctx->N;
    hdr->replicas = replicas;
    hdr->step = ctx->st_step;
    hdr->replica_base = (uint64_t)ctx->st_base;
    uint8_t *p = static_cast<uint8_t *>(buf) + sizeof(da_state_header);
    hipStream_t s = ctx->own_stream;
    uint8_t *x = p, *bx = p + R * N;
    int32_t *h = reinterpret_cast<int32_t *>(p + 2 * R * N);
    uint8_t *tail = p + 6 * R * N;
    hipError_t e = hipMemcpy2DAsync(x, N, ctx->st.x, ld, N, R, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipMemcpy2DAsync(bx, N, ctx->st.bx, ld, N, R, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipMemcpy2DAsync(h, N * 4, ctx->st.h, ld * 4, N * 4, R, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(tail, ctx->st.E, R * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(tail + R * 8, ctx->st.bE, R * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(tail + R * 16, ctx->st.nacc, R * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(tail + R * 24, ctx->st.eoff, R * 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    return check_hip(ctx, e, "state copy to host");
}

int da_state_load(da_ctx *ctx, const void *buf, size_t bytes) {
    if (!ctx || !buf) return fail(ctx, DA_EINVAL, "null argument");
    if (bytes < sizeof(da_state_header)) return fail(ctx, DA_EINVAL, "buffer too short");
    const auto *hdr = static_cast<const da_state_header *>(buf);
    if (hdr->magic != 0x54534144u || hdr->version != 1)
        return fail(ctx, DA_EINVAL, "not a version-1 state snapshot");
    if (hdr->N != ctx->N) return fail(ctx, DA_EINVAL, "snapshot is of a different N");
    if (hdr->replicas < 1 || hdr->step < 0 || hdr->step > kMaxSteps ||
        hdr->replica_base + (uint64_t)hdr->replicas > (uint64_t(1) << 31))
        return fail(ctx, DA_EINVAL, "corrupt snapshot header");
    const int64_t need = da_state_bytes(hdr->N, hdr->replicas);
    if ((int64_t)bytes < need) return fail(ctx, DA_EINVAL, "buffer shorter than the snapshot");
    {
        // the step kernel keeps E_offset in [0, 2^30]; a snapshot outside is corrupt
        const size_t R = (size_t)hdr->replicas, N = (size_t)hdr->N;
        const uint8_t *eo = static_cast<const uint8_t *>(buf) + sizeof(da_state_header) +
                            6 * R * N + 24 * R;
        for (size_t r = 0; r < R; ++r) {
            int32_t v;
            std::memcpy(&v, eo + 4 * r, 4);
            if (v < 0 || v > kEoffMax) return fail(ctx, DA_EINVAL, "snapshot offset out of range");
        }
    }
    std::string err;
    ctx->st_step = -1;
    if (!ctx->st.ensure(hdr->replicas, ctx->ld, err)) return fail(ctx, DA_ENOMEM, err);
    const size_t N = (size_t)ctx->N, ld = (size_t)ctx->ld, R = (size_t)hdr->replicas;
    const uint8_t *p = static_cast<const uint8_t *>(buf) + sizeof(da_state_header);
    const uint8_t *x = p, *bx = p + R * N, *h = p + 2 * R * N, *tail = p + 6 * R * N;
    hipStream_t s = ctx->own_stream;
    // padding columns of the state rows are zero, as the initialisers leave them
    hipError_t e = hipMemsetAsync(ctx->st.x, 0, R * ld, s);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->st.bx, 0, R * ld, s);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->st.h, 0, R * ld * 4, s);
    if (e == hipSuccess) e = hipMemcpy2DAsync(ctx->st.x, ld, x, N, N, R, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpy2DAsync(ctx->st.bx, ld, bx, N, N, R, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpy2DAsync(ctx->st.h, ld * 4, h, N * 4, N * 4, R, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(ctx->st.E, tail, R * 8, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ctx->st.bE, tail + R * 8, R * 8, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ctx->st.nacc, tail + R * 16, R * 8, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ctx->st.eoff, tail + R * 24, R * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    int rc = check_hip(ctx, e, "state upload");
    if (rc) return rc;
    ctx->st_step = hdr->step;
    ctx->st_base = (int64_t)hdr->replica_base;
    ctx->st_R = hdr->replicas;
    return DA_OK;
}

int da_anneal_batch(const da_batch_item *items, int32_t count, void *stream) {
    if (!items || count < 1) return fail(nullptr, DA_EINVAL, "empty batch");
    hipStream_t s = stream ? reinterpret_cast<hipStream_t>(stream) : nullptr;
    for (int32_t a = 0; a < count; ++a)
        for (int32_t c = a + 1; c < count; ++c)
            if (items[a].ctx == items[c].ctx)
                return fail(nullptr, DA_EINVAL, "batch items must use distinct contexts");
    std::vector<JobDesc> jobs((size_t)count);
    std::vector<JobTables> keep((size_t)count);
    // no context claims a resumable state until the whole batch has run
    for (int32_t a = 0; a < count; ++a)
        if (items[a].ctx) items[a].ctx->st_step = -1;
    for (int32_t a = 0; a < count; ++a) {
        const da_batch_item &it = items[a];
        da_ctx *ctx = it.ctx;
        if (!ctx) return fail(nullptr, DA_EINVAL, "batch item without context");
        if (!s) s = ctx->own_stream;
        std::string err;
        int rc = validate_schedule(&it.schedule, err);
        if (rc) return fail(ctx, rc, err);
        if (it.replicas < 1 || it.steps < 0 || it.steps > kMaxSteps || it.replica_base < 0 ||
            it.replica_base + it.replicas > (int64_t(1) << 31))
            return fail(ctx, DA_EINVAL, "bad replicas / steps / replica_base in batch item");
        const LaunchShape sh = batch_shape(ctx, it.replicas, it.schedule);
        JobTables &jt = keep[(size_t)a];
        rc = job_tables(it.schedule, it.steps, sh.wave, jt, err);
        if (rc) return fail(ctx, rc, err);
        ctx->keep_tables = jt.levels;
        ctx->keep_temps = jt.temps;
        if (!ctx->st.ensure(it.replicas, ctx->ld, err)) return fail(ctx, DA_ENOMEM, err);
        jobs[(size_t)a] = make_job(ctx, jt.levels.get(), it.replicas, (uint32_t)it.replica_base,
                                   it.seed, it.steps, it.schedule, sh);
        attach_tables(jobs[(size_t)a], it.schedule, jt);
        if (const char *why = job_range_error(jobs[(size_t)a])) return fail(ctx, DA_EINVAL, why);
        rc = init_state(ctx, jobs[(size_t)a], it.schedule.init, s);
        if (rc) return rc;
    }
    da_ctx *c0 = items[0].ctx;
    // process-lifetime runner (never destroyed: no device frees at exit)
    static std::mutex runner_mu;
    static BatchRunner *runner_p = new BatchRunner();
    BatchRunner &runner = *runner_p;
    std::lock_guard<std::mutex> lock(runner_mu);
    std::string err;
    hipEvent_t be0 = nullptr, be1 = nullptr;
    int rc = next_events(c0, be0, be1);
    if (!rc) rc = check_hip(c0, hipEventRecord(be0, s), "event record");
    if (!rc) {
        rc = runner.run(jobs, s, err);
        if (rc) fail(c0, rc, err);
    }
    for (int32_t a = 0; a < count && !rc; ++a)
        record_stats(items[a].ctx, runner.shapes[(size_t)a], 1, runner.shapes[(size_t)a].gen);
    if (!rc) rc = check_hip(c0, hipEventRecord(be1, s), "event record");
    for (int32_t a = 0; a < count && !rc; ++a)
        rc = extract_outputs(items[a].ctx, jobs[(size_t)a], items[a].replicas, &items[a].out_dev, s);
    // descriptor tables are reused by the next batch: finish this one first, also
    // where it failed on the way
    const hipError_t done = hipStreamSynchronize(s);
    if (!rc) rc = check_hip(c0, done, "stream synchronise");
    if (rc) return rc;
    for (int32_t a = 0; a < count; ++a) {
        da_ctx *ctx = items[a].ctx;
        ctx->st_step = items[a].steps;
        ctx->st_base = items[a].replica_base;
        ctx->st_R = items[a].replicas;
    }
    return DA_OK;
}

}  // extern "C"

namespace {

int check_pt_args(da_ctx *ctx, const double *temps, int32_t M, int32_t chains, int64_t rounds,
                  int32_t steps_per_round, int32_t eoff_inc) {
    if (!temps || M < 1 || M > kMaxLevels || chains < 1 || rounds < 0 || steps_per_round < 0 ||
        eoff_inc < 0)
        return fail(ctx, DA_EINVAL, "bad PT arguments");
    if ((int64_t)M * chains > (int64_t(1) << 30)) return fail(ctx, DA_EINVAL, "too many replicas");
    if (rounds * (int64_t)steps_per_round > kMaxSteps || rounds > kMaxSteps)
        return fail(ctx, DA_EINVAL, "rounds * steps_per_round must be < 2^31");
    for (int p = 0; p < M; ++p) {
        if (!(temps[p] > 0.0) || !std::isfinite(temps[p]))
            return fail(ctx, DA_EINVAL, "temperatures must be finite and > 0");
        if (p + 1 < M && !(temps[p] < temps[p + 1]))
            return fail(ctx, DA_EINVAL, "temperatures must be strictly increasing");
    }
    return DA_OK;
}

// One PT run on the device (arguments already checked): random starts, then
// `rounds` rounds of steps_per_round DA steps and an exchange sweep.
int pt_run(da_ctx *ctx, const double *temps, int32_t M, int32_t chains, int64_t rounds,
           int32_t steps_per_round, int32_t eoff_inc, uint64_t seed, da_pt_result *out) {
    const int32_t R = M * chains;
    const int32_t npair = chains * std::max(M - 1, 1);
    std::string err;
    std::vector<double> tv(temps, temps + M);
    LaunchShape sh;
    const bool wave = wave_shape(ctx, R, temps[0], temps[M - 1], sh);
    JobTables jt;
    if (wave) {
        jt.temps = get_temp_list(tv, err);
        if (!jt.temps || !device_bound_error(jt.gerr, err)) return fail(ctx, DA_ENOMEM, err);
    } else {
        jt.levels = get_level_tables(tv, err);
        if (!jt.levels) return fail(ctx, DA_ENOMEM, err);
    }
    jt.G = device_neg_log_u(err);
    if (!jt.G) return fail(ctx, DA_ENOMEM, err);
    const LevelTables *lt = jt.levels.get();
    ctx->keep_tables = jt.levels;
    ctx->keep_temps = jt.temps;
    ctx->st_step = -1;   // PT state is not a resumable anneal
    if (!ctx->st.ensure(R, ctx->ld, err)) return fail(ctx, DA_ENOMEM, err);
    hipStream_t s = ctx->own_stream;
    int rc = DA_OK;
    if (R > ctx->pt_cap_R || M > ctx->pt_cap_M || chains > ctx->pt_cap_chains ||
        npair > ctx->pt_cap_pairs) {
        for (void *p : {(void *)ctx->pt_slot2rep, (void *)ctx->pt_lvl, (void *)ctx->pt_swaps,
                        (void *)ctx->pt_pair, (void *)ctx->pt_round, (void *)ctx->pt_dbeta})
            if (p) (void)hipFree(p);
        ctx->pt_slot2rep = ctx->pt_lvl = nullptr;
        ctx->pt_swaps = ctx->pt_pair = nullptr;
        ctx->pt_round = nullptr;
        ctx->pt_dbeta = nullptr;
        ctx->pt_cap_R = ctx->pt_cap_M = ctx->pt_cap_chains = ctx->pt_cap_pairs = 0;
        rc = check_hip(ctx, hipMalloc(&ctx->pt_slot2rep, (size_t)R * 4), "PT allocation");
        if (!rc) rc = check_hip(ctx, hipMalloc(&ctx->pt_lvl, (size_t)R * 4), "PT allocation");
        if (!rc) rc = check_hip(ctx, hipMalloc(&ctx->pt_swaps, (size_t)chains * 8), "PT allocation");
        if (!rc) rc = check_hip(ctx, hipMalloc(&ctx->pt_pair, (size_t)npair * 8), "PT allocation");
        if (!rc) rc = check_hip(ctx, hipMalloc(&ctx->pt_round, 8 + (size_t)chains * 4), "PT allocation");
        if (!rc) rc = check_hip(ctx, hipMalloc(&ctx->pt_dbeta, (size_t)M * 8), "PT allocation");
        if (rc) return rc;
        ctx->pt_cap_R = R;
        ctx->pt_cap_M = M;
        ctx->pt_cap_chains = chains;
        ctx->pt_cap_pairs = npair;
    }
    // exchange tables: 1/T_p - 1/T_{p+1}, and -ln U_u
    std::vector<double> dbeta((size_t)M, 0.0);
    for (int p = 0; p + 1 < M; ++p) dbeta[(size_t)p] = 1.0 / temps[p] - 1.0 / temps[p + 1];
    rc = check_hip(ctx, hipMemcpyAsync(ctx->pt_dbeta, dbeta.data(), (size_t)M * 8, hipMemcpyHostToDevice, s), "PT upload");
    if (rc) return rc;

    da_schedule sched{temps[0], temps[0], DA_SCHED_GEOMETRIC, 1, eoff_inc, DA_INIT_RANDOM,
                      DA_TRIAL_PARALLEL, 0};
    if (!wave) sh = choose_shape(ctx, R, nullptr, false);
    JobDesc J = make_job(ctx, lt, R, 0u, seed, 0, sched, sh);
    attach_tables(J, sched, jt);
    // per-draw estimates (one replica per workgroup, several compute waves,
    // fields of many coupling units, as for anneals; the levels' windows are
    // measured when the tables are made): handed over by the random-number
    // waves, whose ring then needs its estimate part in LDS, or evaluated by
    // the compute lanes themselves
    const bool wide16 = ctx->dtype != 2 || (ctx->wscale < (1 << 15) && ctx->wscale > -(1 << 15));
    J.gth = (!wave && lt->any_gth && sh.RPW == 1 && sh.NW > 1 && sh.F >= 4 && !sh.w_lds && wide16 &&
             ctx->ell_D == 0 && ctx->hbound <= kGenFieldMax &&
             ctx->hbound >= 4096 * (int64_t)std::abs(ctx->wscale))
                ? 1
                : 0;
    if (J.gth && sh.NH > 0) {
        const size_t lg = run_lds_bytes(sh.NW, sh.RPW, sh.F, 0, 1, sh.NH, false, false, true);
        if (lg <= (size_t)device_lds_limit()) sh.lds = lg;
        else J.gth = 0;
    }
    J.L = M;
    J.lvl_of_rep = ctx->pt_lvl;
    J.round_ptr = ctx->pt_round;
    J.K = steps_per_round;
    // the wave and team kernels sweep the chains themselves
    const bool sweeps = wave && M <= 64 && steps_per_round > 0;
    if (sweeps)
        J.pt = PtDesc{M, chains, ctx->pt_slot2rep, ctx->pt_lvl, ctx->pt_dbeta, ctx->pt_swaps,
                      ctx->pt_pair, ctx->pt_round, ctx->pt_round + 2};
    if (const char *why = job_range_error(J)) return fail(ctx, DA_EINVAL, why);
    rc = init_state(ctx, J, DA_INIT_RANDOM, s);
    if (!rc)
        rc = check_hip(ctx, (hipError_t)launch_pt_setup(ctx->pt_slot2rep, ctx->pt_lvl,
                                                        ctx->pt_swaps, ctx->pt_pair,
                                                        ctx->pt_round, M, chains, s),
                       "PT setup");
    hipEvent_t pe0 = nullptr, pe1 = nullptr;
    if (!rc) rc = next_events(ctx, pe0, pe1);
    if (!rc) rc = check_hip(ctx, hipEventRecord(pe0, s), "event record");
    if (rc) return rc;

    auto one_round = [&]() -> int {
        int e = 0;
        if (steps_per_round > 0)
            e = wave ? launch_wave(J, sh.F, sh.blocks, sh.threads, sh.lds, s)
                     : launch_run(J, sh.F, sh.NH > 0, nullptr, sh.blocks, sh.threads, sh.lds, s);
        if (!e && !sweeps)
            e = launch_pt_exchange(J.E, ctx->pt_slot2rep, ctx->pt_lvl, ctx->pt_dbeta, jt.G,
                                   M, chains, seed, ctx->pt_round, ctx->pt_swaps, ctx->pt_pair, s);
        return e;
    };
    // Rounds are captured into a hipGraph (kernels only, no memsets) and
    // replayed; each kernel reads the round index from the device counter.
    const int64_t G = std::min<int64_t>(rounds, 32);
    int64_t done = 0;
    if (G >= 2 && rounds >= 2 * G) {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        rc = check_hip(ctx, hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal), "graph capture");
        for (int64_t q = 0; q < G && !rc; ++q) rc = check_hip(ctx, (hipError_t)one_round(), "PT round launch");
        hipError_t ee = hipStreamEndCapture(s, &graph);
        if (!rc) rc = check_hip(ctx, ee, "graph capture end");
        if (!rc) rc = check_hip(ctx, hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0), "graph instantiate");
        for (; !rc && done + G <= rounds; done += G)
            rc = check_hip(ctx, hipGraphLaunch(exec, s), "graph launch");
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (rc) return rc;
    }
    for (; done < rounds && !rc; ++done) rc = check_hip(ctx, (hipError_t)one_round(), "PT round launch");
    if (!rc) rc = check_hip(ctx, hipEventRecord(pe1, s), "event record");
    if (rc) return rc;
    record_stats(ctx, sh, 1, wave ? 1 : J.gth);

    if (out) {
        da_result o{out->best_x, out->best_E, out->final_x, out->final_E, out->n_accept};
        // (a round's fields serve nothing once it is over)
        rc = copy_outputs_to_host(ctx, J, R, &o, s, J.h, (size_t)R * (size_t)J.ld * 4);
        hipError_t e = hipSuccess;
        if (!rc && out->slot) e = hipMemcpy(out->slot, ctx->pt_lvl, (size_t)R * 4, hipMemcpyDeviceToHost);
        if (e == hipSuccess && !rc && out->n_swaps)
            e = hipMemcpy(out->n_swaps, ctx->pt_swaps, (size_t)chains * 8, hipMemcpyDeviceToHost);
        if (e == hipSuccess && !rc && out->pair_swaps && M > 1)
            e = hipMemcpy(out->pair_swaps, ctx->pt_pair, (size_t)chains * (M - 1) * 8,
                          hipMemcpyDeviceToHost);
        if (!rc) rc = check_hip(ctx, e, "PT output copy");
    } else {
        rc = check_hip(ctx, hipStreamSynchronize(s), "stream synchronise");
    }
    return rc;
}

}  // namespace

extern "C" {

int da_pt(da_ctx *ctx, const double *temps, int32_t M, int32_t chains, int64_t rounds,
          int32_t steps_per_round, int32_t eoff_inc, uint64_t seed, da_pt_result *out) {
    if (!ctx) return fail(nullptr, DA_EINVAL, "ctx is null");
    const int rc = check_pt_args(ctx, temps, M, chains, rounds, steps_per_round, eoff_inc);
    if (rc) return rc;
    return pt_run(ctx, temps, M, chains, rounds, steps_per_round, eoff_inc, seed, out);
}

int da_pt_ladder_update(int32_t M, const double *temps, const int64_t *accepted,
                        int64_t proposals, double *out) {
    if (!temps || !out || (M > 1 && !accepted) || M < 1 || proposals < 0)
        return fail(nullptr, DA_EINVAL, "bad ladder-update arguments");
    for (int p = 0; p < M; ++p) out[p] = temps[p];
    if (M < 3 || proposals < 1) return DA_OK;
    // in inverse temperature: the span beta_0 - beta_{M-1} stays, and each
    // pair's interval becomes proportional to (its interval) * (its
    // acceptance, floored at half a swap), so more-accepting pairs widen
    const double beta_cold = 1.0 / temps[0];
    const double beta_hot = 1.0 / temps[M - 1];
    const double floor_acc = 0.5 / (double)proposals;
    std::vector<double> w((size_t)M - 1);
    double total = 0.0;
    for (int p = 0; p + 1 < M; ++p) {
        double a = (double)accepted[p] / (double)proposals;
        if (a < floor_acc) a = floor_acc;
        w[(size_t)p] = (1.0 / temps[p] - 1.0 / temps[p + 1]) * a;
        total += w[(size_t)p];
    }
    double beta = beta_cold;
    for (int p = 0; p + 2 < M; ++p) {
        beta = beta - (beta_cold - beta_hot) * (w[(size_t)p] / total);
        out[p + 1] = 1.0 / beta;
    }
    return DA_OK;
}

int da_pt_adapt(da_ctx *ctx, double *temps, int32_t M, int32_t chains, int32_t iterations,
                int64_t rounds, int32_t steps_per_round, int32_t eoff_inc, uint64_t seed,
                double *acceptance) {
    if (!ctx) return fail(nullptr, DA_EINVAL, "ctx is null");
    if (M < 2 || iterations < 0 || rounds < 1)
        return fail(ctx, DA_EINVAL, "ladder adaptation needs M >= 2, rounds >= 1");
    int rc = check_pt_args(ctx, temps, M, chains, rounds, steps_per_round, eoff_inc);
    if (rc) return rc;
    std::vector<int64_t> ps((size_t)chains * (M - 1)), acc((size_t)M - 1);
    std::vector<double> next((size_t)M);
    const int64_t proposals = (int64_t)chains * rounds;
    for (int32_t it = 0; it < iterations; ++it) {
        da_pt_result o{};
        o.pair_swaps = ps.data();
        rc = pt_run(ctx, temps, M, chains, rounds, steps_per_round, eoff_inc,
                    seed + (uint64_t)it, &o);
        if (rc) return rc;
        for (int p = 0; p + 1 < M; ++p) {
            int64_t a = 0;
            for (int32_t c = 0; c < chains; ++c) a += ps[(size_t)c * (M - 1) + p];
            acc[(size_t)p] = a;
            if (acceptance)
                acceptance[(size_t)it * (M - 1) + p] = (double)a / (double)proposals;
        }
        rc = da_pt_ladder_update(M, temps, acc.data(), proposals, next.data());
        if (rc) return rc;
        for (int p = 0; p < M; ++p) temps[p] = next[(size_t)p];
    }
    return DA_OK;
}

int da_energy(da_ctx *ctx, const uint8_t *x, int32_t count, int64_t *E) {
    if (!ctx || !x || !E || count < 1) return fail(ctx, DA_EINVAL, "bad energy arguments");
    const size_t bytes = (size_t)count * (size_t)ctx->N;
    const JobDesc J = matrix_job(ctx);
    const int planes = coupling_planes(ctx->dtype, ctx->hbound, ctx->wscale);
    const size_t scratch = (size_t)energy_scratch_elems(J, planes, count);
    uint8_t *dX = nullptr;
    int64_t *dE = nullptr, *dS = nullptr;
    hipStream_t s = ctx->own_stream;
    int rc = check_hip(ctx, hipMalloc(&dX, bytes), "energy allocation");
    if (!rc) rc = check_hip(ctx, hipMalloc(&dE, (size_t)count * 8), "energy allocation");
    if (!rc && scratch) rc = check_hip(ctx, hipMalloc(&dS, scratch * 8), "energy allocation");
    if (!rc) rc = check_hip(ctx, hipMemcpyAsync(dX, x, bytes, hipMemcpyHostToDevice, s), "energy upload");
    if (!rc) rc = check_hip(ctx, (hipError_t)launch_energy(J, planes, dX, count, dE, dS, s), "energy launch");
    if (!rc) rc = check_hip(ctx, hipMemcpyAsync(E, dE, (size_t)count * 8, hipMemcpyDeviceToHost, s), "energy copy");
    if (!rc) rc = check_hip(ctx, hipStreamSynchronize(s), "stream synchronise");
    if (dX) (void)hipFree(dX);
    if (dE) (void)hipFree(dE);
    if (dS) (void)hipFree(dS);
    return rc;
}

int da_last_kernel_stats(da_ctx *ctx, da_kernel_stats *stats) {
    if (!ctx || !stats) return fail(ctx, DA_EINVAL, "null argument");
    if (!ctx->have_stats || ctx->ev_used == 0) return fail(ctx, DA_EINVAL, "no launch recorded yet");
    int rc = check_hip(ctx, hipEventSynchronize(ctx->ev1), "event synchronise");
    if (rc) return rc;
    double total = 0.0;
    float ms = 0.f;
    for (size_t q = 0; q < ctx->ev_used; ++q) {
        rc = check_hip(ctx, hipEventElapsedTime(&ms, ctx->ev_pool[q].first, ctx->ev_pool[q].second),
                       "event elapsed time");
        if (rc) return rc;
        total += ms;
    }
    ctx->last.kernel_ms = ms;
    ctx->last.total_ms = total + ctx->folded_ms;
    ctx->last.launches = (int64_t)ctx->ev_used + ctx->folded_calls;
    *stats = ctx->last;
    return DA_OK;
}

int da_reset_kernel_stats(da_ctx *ctx) {
    if (!ctx) return fail(nullptr, DA_EINVAL, "ctx is null");
    if (ctx->ev1) {
        const int rc = check_hip(ctx, hipEventSynchronize(ctx->ev1), "event synchronise");
        if (rc) return rc;
    }
    ctx->ev_used = 0;
    ctx->folded_ms = 0.0;
    ctx->folded_calls = 0;
    return DA_OK;
}

const char *da_last_error(const da_ctx *ctx) {
    if (ctx) return ctx->err.c_str();
    return t_err.c_str();
}

#ifndef DAPT_BUILD_ID
#define DAPT_BUILD_ID "unknown"
#endif
const char *da_build_id(void) { return DAPT_BUILD_ID; }

const char *da_strerror(int status) {
    switch (status) {
        case DA_OK: return "ok";
        case DA_EINVAL: return "invalid argument";
        case DA_ERANGE: return "coefficients out of range";
        case DA_ENOMEM: return "out of memory";
        case DA_EDEVICE: return "device error";
        case DA_ENOTREADY: return "not ready";
        case DA_ENOTFOUND: return "unknown ticket";
        default: return "unknown status";
    }
}

int da_threshold_table(double T, int32_t *thr) {
    if (!thr) return fail(nullptr, DA_EINVAL, "thr is null");
    build_threshold_table(T, thr);
    return DA_OK;
}

double da_level_temperature(const da_schedule *schedule, int32_t level) {
    if (!schedule) return NAN;
    return schedule_temperature(*schedule, level);
}

}  // extern "C"
