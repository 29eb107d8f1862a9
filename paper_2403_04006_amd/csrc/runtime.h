// Host runtime of the permanent engine: the context (device, workspace,
// launch-geometry cache, error state) and the launch sequences.
#pragma once
#include <hip/hip_runtime.h>

#include <map>
#include <string>
#include <utility>
#include <vector>

#include "../../include/pq.h"
#include "plan.h"
#include "pq_common.h"

namespace pq {
// How the forward and extend-row classes of a many-pattern plan are cut into
// chunks (one wavefront each): aim at num_cu * waves_per_cu * chunks_per_wave
// chunks per class, none shorter than min_chunk time states.  The default
// cuts long uneven jobs finely (a short tail of the longest chunks) while the
// minimum keeps the many short jobs of a sampling run in few chunks.
struct ChunkPolicy {
    int32_t waves_per_cu = 64;
    int32_t chunks_per_wave = 8;
    int32_t min_chunk = 256;
};
// One autotuning decision: the policy kept for a job-list shape, its sweep
// time, the default policy's, and how many candidates were timed (0: taken
// from the table).
struct TuneRecord {
    uint64_t sig = 0;
    ChunkPolicy policy;
    double best_ms = 0.0, default_ms = 0.0;
    int32_t candidates = 0;
    // pq_perm_batched: 1 when the work queue beat the static schedule under
    // the kept policy, 0 when it did not, -1 when not timed
    int32_t queue = -1;
};
}  // namespace pq

struct pq_ctx {
    int device = 0;
    int num_cu = 0;
    int clock_khz = 0;
    std::string last_error;

    // device workspace, grown on demand (hipFree waits for earlier work)
    void* ws = nullptr;
    size_t ws_bytes = 0;
    // one-launch permanents: counts of finished workgroups (lent, see
    // take_tickets; without them permanents take the longer way)
    uint32_t* tickets = nullptr;
    uint32_t ticket_turn = 0;
    // cached many-pattern plans and their device descriptors (many.cpp)
    void* many_cache = nullptr;
    // pinned host staging for descriptor uploads; upload_done marks when the
    // last copy out of it has finished
    void* stage = nullptr;
    size_t stage_bytes = 0;
    hipEvent_t upload_done = nullptr;
    // resident workgroups per CU per (binary, nc); 0 = not yet queried
    int occ[4][pq::kMaxDim + 1] = {};

    // autotuning (pq_autotune_enable): chunk policies of pq_perm_many by
    // job-list shape signature and pq_perm's launch shapes by plan shape
    // signature, and the last decision
    bool autotune = false;
    // pq_perm_many replays a captured HIP graph of its launch sequence
    // (pq_graph_enable)
    bool graphs = false;
    std::vector<pq::TuneRecord> tuned;
    pq::TuneRecord last_tune;
    // resident workgroups per CU of the work-queue and walk kernels, by class
    std::map<int, int> queue_occ;
    // reverse-sweep walk variant (pq_walk_variant, PQ_WALK): 2 (register
    // flip digits - 1) + (quad exchanges through ds_swizzle)
    int walk_variant = pq::kWalkDefaultVariant;
    // which classes pq_perm_batched runs as work queues (pq_queue_mode, PQ_QUEUE)
    int queue_mode = PQ_QUEUE_AUTO;
    // when pq_lhaf fills idle lanes across Gray segments (pq_lhaf_pack,
    // PQ_LHAF_PACK)
    int lhaf_pack = PQ_LHAF_PACK_AUTO;
    // when pq_perm_all_outputs takes its contraction form (pq_all_outputs_gemm,
    // PQ_ALL_GEMM), and that form's state: rocBLAS handle, side streams and
    // the last plan (all.cpp; created on first use)
    int all_gemm = PQ_ALL_GEMM_AUTO;
    void* all_cache = nullptr;

    // fault injection (pq_fault_inject, PQ_FAULT_INJECT): while set, every
    // device allocation (PQ_FAULT_ALLOC) or every launch check
    // (PQ_FAULT_LAUNCH) of this ctx fails as if the runtime had refused it
    int fault = PQ_FAULT_NONE;
    int device_alloc(void** p, size_t bytes, const char* what);

    // cancellation (pq_cancel): a pinned, device-mapped word that the work
    // queue polls between chunks; while it is set, entry points refuse new
    // work with PQ_ECANCELLED
    int32_t* cancel_word = nullptr;
    int32_t* cancel_word_dev = nullptr;
    bool cancelled() const { return cancel_word && __atomic_load_n(cancel_word, __ATOMIC_SEQ_CST) != 0; }
    // start of an entry point that enqueues GPU work: clears the error
    // detail; PQ_ECANCELLED while cancellation is requested
    int begin(const char* name);

    // autotune decisions persisted across processes (PQ_AUTOTUNE_CACHE): the
    // file, and this device's key in it (architecture and CU count)
    std::string tune_cache;
    std::string device_key;
    void tune_cache_load();
    void tune_cache_store(const pq::TuneRecord& rec, const char* kind);

    // pinned, device-mapped status word that kernels validating device-side
    // inputs (the sampler's input modes) mark; read after the stream finishes
    int32_t* status_word = nullptr;
    int32_t* status_word_dev = nullptr;
    int status_reset();   // allocate on first use and clear; PQ_OK or an error

    // sweep timing (pq_profile_enable / pq_profile_read)
    bool profiling = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_used;
    std::vector<hipEvent_t> ev_free;
    hipEvent_t take_event();
    void release_events();

    void clear_error() { last_error.clear(); }
    int fail(int status, const char* fmt, ...);
    int check(hipError_t e, const char* what);
    // workspace of at least `bytes`; nullptr on failure (status set)
    void* workspace(size_t bytes);
    // the same for a form that another one can stand in for: nullptr, the
    // workspace kept as it is and no error, where there is no memory for it
    void* try_workspace(size_t bytes);
    // pinned staging of at least `bytes`, free to overwrite (waits for the
    // previous upload out of it); nullptr on failure
    void* staging(size_t bytes);
    // stream-ordered copy of `bytes` from the staging buffer to device memory
    int upload(void* dst, const void* stage_src, size_t bytes, hipStream_t st);
    void release_all();
    int occupancy(int kind, int nc);
};

void pq_release_many_cache(pq_ctx* ctx);
void pq_release_all_cache(pq_ctx* ctx);
// Validate pq_job descriptions (modes, multiplicities, photon counts, output
// overlap).
int pq_validate_jobs(pq_ctx* ctx, int32_t m, const pq_job* jobs, int32_t njobs);

namespace pq {

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int d) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != d) hipSetDevice(d);
    }
    ~DeviceGuard() {
        if (prev >= 0) hipSetDevice(prev);
    }
};

// Bump allocator over the ctx workspace (256-byte aligned pieces).
struct Carve {
    size_t off = 0;
    size_t take(size_t bytes) {
        size_t o = (off + 255) & ~(size_t)255;
        off = o + bytes;
        return o;
    }
};

// Launch geometry of one forward sweep.
struct Geometry {
    int grid = 1;       // workgroups
    uint32_t waves = 1; // active wavefronts
};
// The sweep splits its time-state range evenly over num_cu * waves_per_cu
// wavefronts (each at least kMinStepsPerWave states).  With `spread`, whole rounds
// of the resident wavefronts, and one round, each at least kSpreadSteps states,
// where that share does not fill one.  The default is two rounds of the
// resident wavefronts: the dispatcher hands the second round's workgroups to
// the CUs that finish their first ones early, which evens out unequal CU and
// XCD speeds that a single round leaves on the critical path.
constexpr int kSweepRounds = 2;
// Sweep kernel kind of a plan (see kernels.h).
int sweep_kind(const Plan& p);
// resident wavefronts per CU of that kernel
int resident_waves(pq_ctx* ctx, const Plan& p, int kind);
// rounds x the resident wavefronts per CU of the plan's sweep kernel
int sweep_waves_per_cu(pq_ctx* ctx, const Plan& p, int rounds = kSweepRounds);
Geometry sweep_geometry(pq_ctx* ctx, const Plan& p, int kind, int waves_per_cu, bool spread);
// Shape signature of a single permanent's launch (kernel kind, sums, digits
// and powers: n and the multiplicity class), for the autotuner's records.
uint64_t single_sig(const Plan& p);
// pq_perm's wavefronts per CU: with autotuning on, the decision recorded for
// the plan's shape if there is one; otherwise the default.
int single_waves_per_cu(pq_ctx* ctx, const Plan& p);

// Device scratch of one permanent's launch sequence: compact matrix (or the
// pair sweep's table), +-2B rows, base sums, the two step tables (mixed radices
// only), the workgroup partials and the lanes' sums and weights (mixed radices
// only), at 256-byte aligned offsets.
struct SingleLayout {
    Geometry geo;
    int kind = 0;
    size_t oB = 0, oR = 0, oBase = 0, oTf = 0, oTb = 0, oP = 0, oL = 0, oLw = 0;
    size_t bytes = 0;
    size_t accept = 0;   // without the lanes' sums: what pq_perm_noalloc measures (pairs: 0)
};
SingleLayout single_layout(pq_ctx* ctx, const Plan& p, int kind, int waves_per_cu, bool spread = true);

// One-launch permanents (k_fused_impl.h): whether a plan takes that form (its
// shape fits, and no other decision is recorded for it), its scratch (the workgroups' sums), and the launch.
bool fused_applies(pq_ctx* ctx, const Plan& p);
size_t fused_bytes(pq_ctx* ctx, const Plan& p);
int run_fused(pq_ctx* ctx, const Plan& p, double* partials, uint32_t* tickets, uint32_t turn, const cplx* U, int64_t ldu, cplx* perm,
              cplx* amp, hipStream_t st, bool timed);

// Full single-permanent sequence (prep, table, sweep, final) on the scratch
// `ws` laid out by `L`; `timed` brackets the sweep with profiling events.
int run_single_at(pq_ctx* ctx, const Plan& p, const SingleLayout& L, char* ws, const cplx* U, int64_t ldu,
                  cplx* perm, cplx* amp, hipStream_t st, bool timed);

// The same on the ctx workspace (grown on demand).  With autotuning on, a
// plan shape without a recorded decision first times the whole sequence
// under its candidate shapes (tune_single) and records the fastest.
int run_single(pq_ctx* ctx, const Plan& p, const cplx* U, int64_t ldu, cplx* perm, cplx* amp,
               hipStream_t st);

// Allocation-free entry point's set-up: resolve the device address of its
// static scratch on the current device (once per device).  PQ_OK or an error.
int noalloc_init(int device);

// A set of kTickets device words that are zero between launches, for one ctx;
// null when noalloc_init failed on this device or none is left.
uint32_t* take_tickets(int device);
void give_tickets(int device, uint32_t* tickets);

}  // namespace pq
