// Host runtime (see runtime.h).
#include "runtime.h"

#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>

#include "../../include/pq.h"
#include "kernels.h"

int pq_ctx::fail(int status, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    last_error = buf;
    return status;
}

int pq_ctx::check(hipError_t e, const char* what) {
    if (fault == PQ_FAULT_LAUNCH) return fail(PQ_EDEVICE, "%s: injected launch failure", what);
    if (e == hipSuccess) return PQ_OK;
    return fail(PQ_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

int pq_ctx::device_alloc(void** p, size_t bytes, const char* what) {
    *p = nullptr;
    if (fault == PQ_FAULT_ALLOC) return fail(PQ_ENOMEM, "%s: injected allocation failure (%zu bytes)", what, bytes);
    if (hipMalloc(p, bytes) != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return fail(PQ_ENOMEM, "%s: hipMalloc(%zu) failed", what, bytes);
    }
    return PQ_OK;
}

int pq_ctx::begin(const char* name) {
    clear_error();
    if (cancelled()) return fail(PQ_ECANCELLED, "%s: cancellation requested on this ctx (pq_cancel)", name);
    return PQ_OK;
}

// One line per decision: {"device": "<arch>:<CUs>", "kind": "<kind>",
// "sig": <decimal>, "policy": [a, b, c], "best_ms": x, "default_ms": y}.
void pq_ctx::tune_cache_load() {
    if (tune_cache.empty()) return;
    FILE* f = fopen(tune_cache.c_str(), "r");
    if (!f) return;
    char line[1024];
    while (fgets(line, sizeof(line), f)) {
        char dev[256] = {0}, kind[64] = {0};
        unsigned long long sig = 0;
        int a = 0, b = 0, c = 0, qd = -1;
        double best = 0.0, def = 0.0;
        const int got = sscanf(line, " {\"device\": \"%255[^\"]\", \"kind\": \"%63[^\"]\", \"sig\": %llu, "
                               "\"policy\": [%d, %d, %d], \"best_ms\": %lf, \"default_ms\": %lf, \"queue\": %d",
                               dev, kind, &sig, &a, &b, &c, &best, &def, &qd);
        if (got < 8) continue;
        if (device_key != dev) continue;
        pq::TuneRecord r;
        r.sig = sig;
        r.policy.waves_per_cu = a;
        r.policy.chunks_per_wave = b;
        r.policy.min_chunk = c;
        r.best_ms = best;
        r.default_ms = def;
        r.candidates = 0;
        r.queue = got == 9 ? qd : -1;
        bool dup = false;
        for (const pq::TuneRecord& t : tuned) dup = dup || t.sig == r.sig;
        if (!dup) tuned.push_back(r);
    }
    fclose(f);
}

void pq_ctx::tune_cache_store(const pq::TuneRecord& rec, const char* kind) {
    if (tune_cache.empty()) return;
    FILE* f = fopen(tune_cache.c_str(), "a");
    if (!f) return;
    fprintf(f, "{\"device\": \"%s\", \"kind\": \"%s\", \"sig\": %llu, \"policy\": [%d, %d, %d], "
            "\"best_ms\": %.6f, \"default_ms\": %.6f, \"queue\": %d}\n", device_key.c_str(), kind,
            (unsigned long long)rec.sig, rec.policy.waves_per_cu, rec.policy.chunks_per_wave, rec.policy.min_chunk,
            rec.best_ms, rec.default_ms, rec.queue);
    fclose(f);
}

// hipFree waits for earlier work that uses the old block
static constexpr size_t kMinWorkspace = (size_t)1 << 20;

void* pq_ctx::workspace(size_t bytes) {
    if (bytes <= ws_bytes && ws) return ws;
    if (ws) {
        hipFree(ws);
        ws = nullptr;
        ws_bytes = 0;
    }
    const size_t want = std::max(bytes, kMinWorkspace);
    if (device_alloc(&ws, want, "workspace")) return nullptr;
    ws_bytes = want;
    return ws;
}

void* pq_ctx::try_workspace(size_t bytes) {
    if (bytes <= ws_bytes && ws) return ws;
    const size_t want = std::max(bytes, kMinWorkspace);
    void* more = nullptr;
    if (device_alloc(&more, want, "workspace")) {
        clear_error();
        return nullptr;
    }
    if (ws) hipFree(ws);
    ws = more;
    ws_bytes = want;
    return ws;
}

hipEvent_t pq_ctx::take_event() {
    if (!ev_free.empty()) {
        hipEvent_t e = ev_free.back();
        ev_free.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

void pq_ctx::release_events() {
    for (auto& pr : ev_used) {
        ev_free.push_back(pr.first);
        ev_free.push_back(pr.second);
    }
    ev_used.clear();
}

void* pq_ctx::staging(size_t bytes) {
    if (upload_done) {
        if (hipEventSynchronize(upload_done) != hipSuccess) {
            fail(PQ_EDEVICE, "staging: wait for previous upload failed");
            return nullptr;
        }
    }
    if (stage && stage_bytes >= bytes) return stage;
    if (stage) hipHostFree(stage);
    stage = nullptr;
    stage_bytes = 0;
    size_t want = bytes < ((size_t)1 << 20) ? ((size_t)1 << 20) : bytes;
    if (hipHostMalloc(&stage, want, hipHostMallocDefault) != hipSuccess) {
        stage = nullptr;
        fail(PQ_ENOMEM, "staging: hipHostMalloc(%zu) failed", want);
        return nullptr;
    }
    stage_bytes = want;
    return stage;
}

int pq_ctx::upload(void* dst, const void* stage_src, size_t bytes, hipStream_t st) {
    if (!upload_done) {
        int rc = check(hipEventCreateWithFlags(&upload_done, hipEventDisableTiming), "upload event");
        if (rc) return rc;
    }
    int rc = check(hipMemcpyAsync(dst, stage_src, bytes, hipMemcpyHostToDevice, st), "upload");
    if (rc) return rc;
    return check(hipEventRecord(upload_done, st), "upload record");
}

int pq_ctx::status_reset() {
    if (!status_word) {
        void* h = nullptr;
        if (hipHostMalloc(&h, 256, hipHostMallocMapped) != hipSuccess)
            return fail(PQ_ENOMEM, "status word: hipHostMalloc failed");
        void* d = nullptr;
        if (hipHostGetDevicePointer(&d, h, 0) != hipSuccess) {
            hipHostFree(h);
            return fail(PQ_EDEVICE, "status word: hipHostGetDevicePointer failed");
        }
        status_word = (int32_t*)h;
        status_word_dev = (int32_t*)d;
    }
    __atomic_store_n(status_word, 0, __ATOMIC_SEQ_CST);
    return PQ_OK;
}

void pq_ctx::release_all() {
    if (cancel_word) hipHostFree(cancel_word);
    cancel_word = nullptr;
    cancel_word_dev = nullptr;
    if (status_word) hipHostFree(status_word);
    status_word = nullptr;
    status_word_dev = nullptr;
    if (upload_done) hipEventDestroy(upload_done);
    upload_done = nullptr;
    if (stage) hipHostFree(stage);
    stage = nullptr;
    stage_bytes = 0;
    release_events();
    for (hipEvent_t e : ev_free) hipEventDestroy(e);
    ev_free.clear();
    if (ws) hipFree(ws);
    ws = nullptr;
    ws_bytes = 0;
    pq::give_tickets(device, tickets);
    tickets = nullptr;
}

int pq_ctx::occupancy(int kind, int nc) {
    int& o = occ[kind][nc];
    if (o == 0) {
        o = kind == pq::kSweepPair ? pq::occupancy_pair(nc) : pq::occupancy_glynn(kind, nc);
        if (o < 1) o = 1;
    }
    return o;
}

namespace pq {

// Fewest time steps per wavefront worth a wavefront's start-up (the column
// sums are rebuilt from the digits, about (digits x NC) multiply-adds).
static constexpr uint64_t kMinStepsPerWave = 32;
// and in a sweep that leaves the device part empty at that share, where a
// wavefront more costs nothing else: 34 photons in 17 modes 36 us at 16, 34 at 8
// and 4; 48 photons in 6 modes 27.8, 20.0 and 16.9
static constexpr uint64_t kSpreadSteps = 4;

// The pair sweep from 2^16 time states on, in three launches against one of the
// one-by-one walk: 22 photons (2^15) 23.3 and 23.0 us a call, 23 30.4 and 33.8,
// 24 44.4 and 51.2; and against its three: 25 photons 79.8 and 108, 26 144 and
// 187.  Beyond 32 columns two wavefronts' registers do not hold the pairs.
static constexpr int kPairTimeDigits = 16;
// Its workgroups: one round of the resident ones, and one for every
// kPairBlocks blocks of eight states (at two rounds of wavefronts; the tuner's
// one and four rounds scale it) where that is more, since equal shares leave the
// fastest of the eight XCDs idle for 6 % of the time: 30 photons at 1024
// workgroups 2.41 ms, 2048 2.38, 8192 2.28, 16384 2.25; but 28 photons 545, 545,
// 562 and 621 us, where the start-up (two blocks' work) shows.
static constexpr uint64_t kPairBlocks = 128;
static constexpr uint64_t kPairMaxGroups = 16384;

int sweep_kind(const Plan& p) {
    if (p.binary)
        return p.nc >= kPairMinCols && p.nc <= kPairMaxCols && p.n_time >= kPairTimeDigits ? kSweepPair : kSweepBin;
    PowSteps ps;
    make_pow_steps(p.col_kap, p.nc, ps);
    return ps.general ? kSweepMixGeneral : kSweepMix;
}

int resident_waves(pq_ctx* ctx, const Plan& p, int kind) {
    return ctx->occupancy(kind, p.nc) * (kind == kSweepPair ? 2 : kWavesPerBlock);
}

int sweep_waves_per_cu(pq_ctx* ctx, const Plan& p, int rounds) {
    return resident_waves(ctx, p, sweep_kind(p)) * rounds;
}

Geometry sweep_geometry(pq_ctx* ctx, const Plan& p, int kind, int waves_per_cu, bool spread) {
    Geometry g;
    const uint64_t full = (uint64_t)(waves_per_cu > 0 ? waves_per_cu : 1) * (uint64_t)ctx->num_cu;
    if (kind == kSweepPair) {
        const uint64_t round = (uint64_t)resident_waves(ctx, p, kind) * (uint64_t)ctx->num_cu / 2;
        const uint64_t rounds = std::max(full / 2 / std::max(round, (uint64_t)1), (uint64_t)1);
        const uint64_t blocks = p.time_states >> 3;
        const uint64_t groups = std::min(std::max(round, blocks * rounds / (2 * kPairBlocks)), kPairMaxGroups);
        g.grid = (int)std::max(std::min(groups, blocks), (uint64_t)1);
        g.waves = 2 * (uint32_t)g.grid;
        return g;
    }
    const uint64_t round = (uint64_t)resident_waves(ctx, p, kind) * (uint64_t)ctx->num_cu;
    uint64_t waves = (p.time_states + kMinStepsPerWave - 1) / kMinStepsPerWave;
    if (waves > full) waves = full;
    if (!spread) {
        // the share alone
    } else if (waves > round) {
        // whole rounds: one begun for a few wavefronts costs a whole one
        // (2 x 15 rows, 1.08 rounds: 83 us, one round: 74)
        waves = waves / round * round;
    } else {
        // too short for a full round at that share: spread over one
        waves = (p.time_states + kSpreadSteps - 1) / kSpreadSteps;
        if (waves > round) waves = round;
        if (waves > full) waves = full;
    }
    if (waves < 1) waves = 1;
    g.waves = (uint32_t)waves;
    g.grid = (int)((waves + kWavesPerBlock - 1) / kWavesPerBlock);
    return g;
}

// Time states up to which a permanent takes one launch, and its wavefronts'
// least share of them (two workgroups per CU at most).  Whole calls, several
// launches -> one: 8 photons 19.2 -> 13.3 us, 16 20.9 -> 15.2, 20 24.0 -> 16.5, 22
// 33.4 -> 23.0 (23 and more go by pairs, kPairTimeDigits); 2 x 9 rows 19.7 -> 13.2,
// 2 x 11 19.9 -> 15.9, 2 x 12 (6,561 states) 20.0 -> 19.7; but 27 photons in 17
// modes (13,824) 20.6 -> 23.8, 2 x 13 (19,683) 21.6 -> 27.6, where the step table
// of the longer sweep is the cheaper step.  Shares of 4, 8 and 16 states: 20
// photons 19.4, 16.5, 16.3 us; 2 x 9 rows 13.7, 16.7, 21.8.
constexpr uint64_t kFusedMaxBinary = 1 << 15;
constexpr uint64_t kFusedMaxMixed = 1 << 13;
constexpr uint64_t kFusedSteps = 8;
constexpr uint64_t kFusedStepsMixed = 4;

static bool fused_shape(const Plan& p) {
    return p.nc <= kFusedMaxCols && p.time_states <= (p.binary ? kFusedMaxBinary : kFusedMaxMixed) &&
           sweep_kind(p) != kSweepMixGeneral;
}

uint64_t single_sig(const Plan& p) {
    // seeded apart from the job-list shape signatures, which share the
    // records and the cache file
    uint64_t h = 0x70657266ull * 1099511628211ull;
    auto mix = [&](uint64_t x) {
        h ^= x;
        h *= 1099511628211ull;
        h ^= h >> 29;
    };
    // (shapes that the one-launch form may take apart from records made without it)
    mix((uint64_t)sweep_kind(p) + (fused_shape(p) ? 16 : 0));
    mix((uint64_t)p.r);
    mix((uint64_t)p.nc);
    mix((uint64_t)p.n_lane);
    for (int k = 0; k < p.n_lane; ++k) mix((uint64_t)p.lane_radix[k]);
    mix((uint64_t)p.n_time);
    for (int k = 0; k < p.n_time; ++k) mix((uint64_t)p.time_radix[k]);
    mix((uint64_t)p.n_inner);
    for (int j = 0; j < p.nc; ++j) mix((uint64_t)p.col_kap[j]);
    return h;
}

static const TuneRecord* recorded(pq_ctx* ctx, uint64_t sig) {
    for (const TuneRecord& t : ctx->tuned)
        if (t.sig == sig) return &t;
    return nullptr;
}

int single_waves_per_cu(pq_ctx* ctx, const Plan& p) {
    if (ctx->autotune)
        if (const TuneRecord* t = recorded(ctx, single_sig(p)))
            if (t->policy.waves_per_cu > 0) return t->policy.waves_per_cu;
    return sweep_waves_per_cu(ctx, p);
}

// `launch()`, bracketed by timing events when `timed` and profiling is on.
template <class F>
static int timed_sweep(pq_ctx* ctx, bool timed, hipStream_t st, F launch) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    timed = timed && ctx->profiling;
    if (timed) {
        e0 = ctx->take_event();
        e1 = ctx->take_event();
        if (!e0 || !e1) return ctx->fail(PQ_EDEVICE, "profile: hipEventCreate failed");
        int rc = ctx->check(hipEventRecord(e0, st), "profile: record");
        if (rc) return rc;
    }
    int rc = ctx->check(launch(), "sweep");
    if (rc) return rc;
    if (timed) {
        rc = ctx->check(hipEventRecord(e1, st), "profile: record");
        if (rc) return rc;
        ctx->ev_used.emplace_back(e0, e1);
    }
    return PQ_OK;
}

// A recorded launch shape of 0 wavefronts per CU is the one-launch form.
bool fused_applies(pq_ctx* ctx, const Plan& p) {
    if (!ctx->tickets || !fused_shape(p)) return false;
    const TuneRecord* t = ctx->autotune ? recorded(ctx, single_sig(p)) : nullptr;
    return !t || t->policy.waves_per_cu <= 0;
}

static uint32_t fused_waves(pq_ctx* ctx, const Plan& p) {
    const uint64_t most = (uint64_t)ctx->num_cu * 2 * kWavesPerBlock;
    const uint64_t least = p.binary ? kFusedSteps : kFusedStepsMixed;
    uint64_t waves = (p.time_states + least - 1) / least;
    if (waves > most) waves = most;
    return (uint32_t)(waves < 1 ? 1 : waves);
}

size_t fused_bytes(pq_ctx* ctx, const Plan& p) {
    return sizeof(double) * 4 * (size_t)((fused_waves(ctx, p) + kWavesPerBlock - 1) / kWavesPerBlock);
}

int run_fused(pq_ctx* ctx, const Plan& p, double* partials, uint32_t* tickets, uint32_t turn, const cplx* U, int64_t ldu, cplx* perm,
              cplx* amp, hipStream_t st, bool timed) {
    FusedArgs a;
    memset(&a, 0, sizeof(a));
    a.U = U;
    a.ldu = ldu;
    a.perm = perm;
    a.amp = amp;
    a.scale = p.scale;
    a.norm = p.norm;
    a.partials = partials;
    a.tickets = tickets;
    a.turn = turn % kTickets;
    a.time_states = (uint32_t)p.time_states;
    a.waves = fused_waves(ctx, p);
    a.r = p.r;
    a.nc = p.nc;
    a.transposed = p.transposed;
    a.n_lane = p.n_lane;
    a.lane_states = p.lane_states;
    a.n_time = p.n_time;
    for (int i = 0; i < p.r; ++i) {
        a.row_mode[i] = p.row_mode[i];
        a.row_mu[i] = (int8_t)p.row_mu[i];
        a.radix[i] = (int8_t)p.row_radix[i];
    }
    for (int j = 0; j < p.nc; ++j) a.col_mode[j] = p.col_mode[j];
    // the padded column repeats the largest power
    int kap[kFusedMaxCols];
    const int nc = (p.nc + 1) / 2 * 2;
    for (int j = 0; j < nc; ++j) kap[j] = p.col_kap[j < p.nc ? j : p.nc - 1];
    make_pow_steps(kap, nc, a.pw);
    const int grid = (int)((a.waves + kWavesPerBlock - 1) / kWavesPerBlock);
    return timed_sweep(ctx, timed, st, [&] { return launch_fused(!p.binary, a, grid, st); });
}

SingleLayout single_layout(pq_ctx* ctx, const Plan& p, int kind, int waves_per_cu, bool spread) {
    SingleLayout L;
    L.geo = sweep_geometry(ctx, p, kind, waves_per_cu, spread);
    L.kind = kind;
    const int r = p.r, nc = p.nc;
    const size_t ntab = p.binary ? 0 : (size_t)p.m_inner;
    Carve cv;
    if (kind == kSweepPair) {
        L.oB = cv.take(sizeof(cplx) * pair_table_size((nc + 1) / 2, p.n_time - 3));
        L.oP = cv.take(sizeof(double) * 4 * (size_t)L.geo.grid);
        L.bytes = cv.off;
        return L;
    }
    L.oB = cv.take(sizeof(cplx) * r * nc);
    L.oR = cv.take(sizeof(cplx) * r * 2 * nc);
    L.oBase = cv.take(sizeof(cplx) * nc);
    L.oTf = cv.take(sizeof(StepEntry) * ntab);
    L.oTb = cv.take(sizeof(StepEntry) * ntab);
    L.oP = cv.take(sizeof(double) * 4 * (size_t)L.geo.grid);
    // (what pq_perm_noalloc accepts was settled without the lanes' sums)
    L.accept = cv.off;
    if (!p.binary) {
        L.oL = cv.take(sizeof(cplx) * 64 * (size_t)nc);
        L.oLw = cv.take(sizeof(double) * 64);
    }
    L.bytes = cv.off;
    return L;
}

static int run_final(pq_ctx* ctx, const Plan& p, const double* partials, int count, cplx* perm, cplx* amp,
                     hipStream_t st) {
    FinalArgs fa;
    fa.partials = partials;
    fa.count = count;
    fa.scale = p.scale;
    fa.norm = p.norm;
    fa.perm = perm;
    fa.amp = amp;
    return ctx->check(launch_final(fa, st), "final");
}

// The pair sweep's launches: table, sweep, final sum.
static int run_pair(pq_ctx* ctx, const Plan& p, const SingleLayout& L, char* ws, const cplx* U, int64_t ldu, cplx* perm,
                    cplx* amp, hipStream_t st, bool timed) {
    PairPrepArgs pa;
    memset(&pa, 0, sizeof(pa));
    pa.U = U;
    pa.ldu = ldu;
    pa.tab = (cplx*)(ws + L.oB);
    pa.r = p.r;
    pa.nc = p.nc;
    pa.pairs = (p.nc + 1) / 2;
    pa.transposed = p.transposed;
    pa.n_lane = p.n_lane;
    pa.n_outer = p.n_time - 3;
    for (int i = 0; i < p.r; ++i) {
        pa.row_mode[i] = p.row_mode[i];
        pa.row_mu[i] = p.row_mu[i];
    }
    for (int j = 0; j < p.nc; ++j) pa.col_mode[j] = p.col_mode[j];
    int rc = ctx->check(launch_pair_prep(pa, st), "pair table");
    if (rc) return rc;
    PairArgs a;
    a.tab = pa.tab;
    a.partials = (double*)(ws + L.oP);
    a.blocks = p.time_states >> 3;
    a.groups = (uint32_t)L.geo.grid;
    a.n_lane = p.n_lane;
    a.lane_states = p.lane_states;
    a.n_outer = pa.n_outer;
    rc = timed_sweep(ctx, timed, st, [&] { return launch_pair(p.nc, a, st); });
    if (rc) return rc;
    return run_final(ctx, p, a.partials, L.geo.grid, perm, amp, st);
}

int run_single_at(pq_ctx* ctx, const Plan& p, const SingleLayout& L, char* ws, const cplx* U, int64_t ldu,
                  cplx* perm, cplx* amp, hipStream_t st, bool timed) {
    if (L.kind == kSweepPair) return run_pair(ctx, p, L, ws, U, ldu, perm, amp, st, timed);
    const int r = p.r, nc = p.nc;
    PrepArgs pa;
    memset(&pa, 0, sizeof(pa));
    pa.U = U;
    pa.ldu = ldu;
    pa.B = (cplx*)(ws + L.oB);
    pa.rows2 = (cplx*)(ws + L.oR);
    pa.base = (cplx*)(ws + L.oBase);
    pa.r = r;
    pa.nc = nc;
    pa.transposed = p.transposed;
    for (int i = 0; i < r; ++i) { pa.row_mode[i] = p.row_mode[i]; pa.row_mu[i] = p.row_mu[i]; }
    for (int j = 0; j < nc; ++j) pa.col_mode[j] = p.col_mode[j];
    if (!p.binary) {
        pa.tab_fwd = (StepEntry*)(ws + L.oTf);
        pa.tab_bwd = (StepEntry*)(ws + L.oTb);
        pa.lane_sums = (cplx*)(ws + L.oL);
        pa.lane_w = (double*)(ws + L.oLw);
        pa.n_inner = p.n_inner;
        pa.m_inner = p.m_inner;
        pa.n_lane = p.n_lane;
        pa.lane_states = p.lane_states;
        for (int k = 0; k < p.n_lane; ++k) pa.lane_radix[k] = p.lane_radix[k];
        for (int k = 0; k < p.n_inner; ++k) pa.radix[k] = p.time_radix[k];
    }
    int rc = ctx->check(launch_prep(pa, st), "prep");
    if (rc) return rc;

    GlynnArgs ga;
    memset(&ga, 0, sizeof(ga));
    ga.B = pa.B;
    ga.rows2 = pa.rows2;
    ga.base = pa.base;
    ga.tab_fwd = (const StepEntry*)(ws + L.oTf);
    ga.tab_bwd = (const StepEntry*)(ws + L.oTb);
    ga.partials = (double*)(ws + L.oP);
    ga.time_states = p.time_states;
    ga.waves = L.geo.waves;
    ga.n_lane = p.n_lane;
    ga.lane_states = p.lane_states;
    ga.n_time = p.n_time;
    ga.n_inner = p.n_inner;
    ga.m_inner = p.m_inner;
    for (int k = 0; k < p.n_lane; ++k) ga.lane_radix[k] = p.lane_radix[k];
    for (int k = 0; k < p.n_time; ++k) {
        ga.time_radix[k] = p.time_radix[k];
        ga.time_inv[k] = digit_inverse((uint32_t)p.time_radix[k]);
    }
    ga.lane_sums = pa.lane_sums;
    ga.lane_w = pa.lane_w;
    for (int j = 0; j < nc; ++j) ga.kap[j] = p.col_kap[j];
    make_pow_steps(ga.kap, nc, ga.pw);

    rc = timed_sweep(ctx, timed, st, [&] { return launch_glynn(L.kind, nc, ga, L.geo.grid, st); });
    if (rc) return rc;
    return run_final(ctx, p, ga.partials, L.geo.grid, perm, amp, st);
}

// Time the whole launch sequence of a plan under 2, 1 and 4 rounds of the
// resident wavefronts (the default first; best of two runs each), and record the
// fastest for the plan's shape.  Where the one-launch form applies, that is the
// default and comes first instead of the 2 rounds (so few states make the same
// launch of any).  The runs write perm and amp; the caller's run afterwards writes
// them again.
static int tune_single(pq_ctx* ctx, const Plan& p, const cplx* U, int64_t ldu, cplx* perm, cplx* amp,
                       hipStream_t st) {
    TuneRecord rec;
    rec.sig = single_sig(p);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) hipEventDestroy(e0);
        return ctx->fail(PQ_EDEVICE, "tune: hipEventCreate failed");
    }
    int rc = PQ_OK;
    double best = -1.0;
    const bool fused = ctx->tickets && fused_shape(p);
    for (int rounds : {kSweepRounds, 1, 4}) {
        const bool one = fused && rec.candidates == 0;
        const int w = one ? 0 : sweep_waves_per_cu(ctx, p, rounds);
        SingleLayout L;
        if (!one) L = single_layout(ctx, p, sweep_kind(p), w);
        char* ws = (char*)ctx->workspace(one ? fused_bytes(ctx, p) : L.bytes);
        if (!ws) {
            rc = PQ_ENOMEM;
            break;
        }
        double ms = -1.0;
        for (int rep = 0; rep < 2 && !rc; ++rep) {
            rc = ctx->check(hipEventRecord(e0, st), "tune: record");
            if (!rc) rc = one ? run_fused(ctx, p, (double*)ws, ctx->tickets, ctx->ticket_turn++, U, ldu, perm, amp, st, false)
                              : run_single_at(ctx, p, L, ws, U, ldu, perm, amp, st, false);
            if (!rc) rc = ctx->check(hipEventRecord(e1, st), "tune: record");
            if (!rc) rc = ctx->check(hipEventSynchronize(e1), "tune: synchronize");
            float f = 0.0f;
            if (!rc) rc = ctx->check(hipEventElapsedTime(&f, e0, e1), "tune: elapsed");
            if (!rc && (ms < 0.0 || f < ms)) ms = f;
        }
        if (rc) break;
        ++rec.candidates;
        if (rec.candidates == 1) rec.default_ms = ms;
        if (best < 0.0 || ms < best) {
            best = ms;
            rec.policy.waves_per_cu = w;
            rec.policy.chunks_per_wave = 1;
            rec.policy.min_chunk = (int32_t)kMinStepsPerWave;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (rc) return rc;
    rec.best_ms = best;
    ctx->tuned.push_back(rec);
    ctx->last_tune = rec;
    ctx->tune_cache_store(rec, "perm");
    return PQ_OK;
}

int run_single(pq_ctx* ctx, const Plan& p, const cplx* U, int64_t ldu, cplx* perm, cplx* amp,
               hipStream_t st) {
    if (ctx->autotune) {
        if (const TuneRecord* t = recorded(ctx, single_sig(p))) {
            ctx->last_tune = *t;
            ctx->last_tune.candidates = 0;
        } else if (int rc = tune_single(ctx, p, U, ldu, perm, amp, st)) {
            return rc;
        }
    }
    if (fused_applies(ctx, p)) {
        double* partials = (double*)ctx->workspace(fused_bytes(ctx, p));
        if (!partials) return PQ_ENOMEM;
        return run_fused(ctx, p, partials, ctx->tickets, ctx->ticket_turn++, U, ldu, perm, amp, st, true);
    }
    const SingleLayout L = single_layout(ctx, p, sweep_kind(p), single_waves_per_cu(ctx, p));
    char* ws = (char*)ctx->workspace(L.bytes);
    if (!ws) return PQ_ENOMEM;
    return run_single_at(ctx, p, L, ws, U, ldu, perm, amp, st, true);
}

}  // namespace pq
