// pq_perm_noalloc: pq_perm for callers that cannot allocate device memory
// (code under HIP graph capture, tight serving loops).  Its launch sequence
// runs on a file-scope device array instead of the ctx workspace.
//
// Host code must not pass `scratch` itself to a kernel: in host code the name
// stands for a host-side shadow, not a device address.  noalloc_init (called
// by pq_create with the device current) resolves the device address once per
// device with hipGetSymbolAddress, and every use goes through that address.
#include <hip/hip_runtime.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <vector>

#include "../../include/pq.h"
#include "kernels.h"
#include "plan.h"
#include "runtime.h"

namespace pq {

// what is accepted, and the buffer, which also holds the pair sweep's sums
constexpr size_t kNoAllocScratchBytes = PQ_NOALLOC_SCRATCH_BYTES;
constexpr size_t kNoAllocBufferBytes = 640 * 1024;
constexpr int kNoAllocMaxDevices = 64;

static __device__ __align__(256) char scratch[kNoAllocBufferBytes];
// the one-launch form's workgroup counts, zero from the start and between
// launches: the first for this file, the others lent to one ctx each
constexpr int kTicketSets = 1024;
static __device__ uint32_t ticket_sets[kTicketSets][kTickets];

static std::mutex g_scratch_mu;
// turns through the first set, over every ctx
static std::atomic<uint32_t> g_noalloc_turn{0};
static std::vector<bool> g_sets_taken[kNoAllocMaxDevices];
static char* g_scratch_dev[kNoAllocMaxDevices] = {};
static uint32_t* g_tickets_dev[kNoAllocMaxDevices] = {};

int noalloc_init(int device) {
    if (device < 0 || device >= kNoAllocMaxDevices) return PQ_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_dev[device]) return PQ_OK;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
        (void)hipGetLastError();
        return PQ_EDEVICE;
    }
    void* tickets = nullptr;
    if (hipGetSymbolAddress(&tickets, HIP_SYMBOL(ticket_sets)) != hipSuccess || !tickets) {
        (void)hipGetLastError();
        return PQ_EDEVICE;
    }
    g_tickets_dev[device] = (uint32_t*)tickets;
    g_scratch_dev[device] = (char*)ptr;
    return PQ_OK;
}

uint32_t* take_tickets(int device) {
    if (device < 0 || device >= kNoAllocMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_tickets_dev[device]) return nullptr;
    std::vector<bool>& taken = g_sets_taken[device];
    taken.resize(kTicketSets, false);
    for (int k = 1; k < kTicketSets; ++k)
        if (!taken[k]) {
            taken[k] = true;
            return g_tickets_dev[device] + (size_t)k * kTickets;
        }
    return nullptr;
}

void give_tickets(int device, uint32_t* tickets) {
    if (!tickets) return;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    g_sets_taken[device][(size_t)(tickets - g_tickets_dev[device]) / kTickets] = false;
}

static char* scratch_of(int device, uint32_t** tickets) {
    if (device < 0 || device >= kNoAllocMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    *tickets = g_tickets_dev[device];
    return g_scratch_dev[device];
}

}  // namespace pq

using namespace pq;

int pq_perm_noalloc(pq_ctx* ctx, const pq_c128* U, int64_t ldu, int32_t m,
                    const int32_t* S, const int32_t* T,
                    pq_c128* perm, pq_c128* amp, void* stream) {
    if (!ctx) return PQ_EINVAL;
    if (int rc_ = ctx->begin("pq_perm_noalloc")) return rc_;
    if (m < 0 || !S || !T) return ctx->fail(PQ_EINVAL, "pq_perm_noalloc: m < 0 or NULL occupation vector");
    if (m > 0 && (!U || ldu < m)) return ctx->fail(PQ_EINVAL, "pq_perm_noalloc: NULL U or ldu < m");
    Plan p;
    plan_dense(m, S, T, p);
    if (p.status != PQ_OK) return ctx->fail(p.status, "pq_perm_noalloc: planning failed (%s)", pq_strerror(p.status));
    DeviceGuard guard(ctx->device);
    hipStream_t st = (hipStream_t)stream;
    if (p.trivial) {
        cplx v = p.trivial == 1 ? cplx{0.0, 0.0} : cplx{1.0, 0.0};
        if (!perm && !amp) return PQ_OK;
        return ctx->check(launch_fill((cplx*)perm, (cplx*)amp, v, st), "fill");
    }
    uint32_t* tickets = nullptr;
    char* ws = scratch_of(ctx->device, &tickets);
    if (!ws) return ctx->fail(PQ_EDEVICE, "pq_perm_noalloc: the static scratch of device %d was not resolved", ctx->device);
    // what fits is decided by the sweep without the spread (its partials can need
    // more scratch); other forms are taken where they fit too.  Every plan of the
    // pair sweep is accepted (accept 0): the buffer holds its table, 73 KB at most,
    // and its most workgroups' sums, 512 KB; and the single columns' sweep that
    // decided before there were pairs needed at most 148 KB of the 160 for these
    // plans under any tuned shape
    const int kind = sweep_kind(p);
    const int wpc = single_waves_per_cu(ctx, p);
    SingleLayout L = single_layout(ctx, p, kind, wpc, false);
    if (L.accept > kNoAllocScratchBytes)
        return ctx->fail(PQ_ERANGE, "pq_perm_noalloc: this permanent needs %zu bytes of scratch, more than the %zu "
                         "bytes of the static buffer (use pq_perm)", L.accept, kNoAllocScratchBytes);
    if (fused_applies(ctx, p) && fused_bytes(ctx, p) <= kNoAllocBufferBytes)
        return run_fused(ctx, p, (double*)ws, tickets, g_noalloc_turn.fetch_add(1), (const cplx*)U, ldu, (cplx*)perm, (cplx*)amp, st, false);
    const SingleLayout spread = single_layout(ctx, p, kind, wpc);
    if (spread.bytes <= kNoAllocBufferBytes) L = spread;
    return run_single_at(ctx, p, L, ws, (const cplx*)U, ldu, (cplx*)perm, (cplx*)amp, st, false);
}
