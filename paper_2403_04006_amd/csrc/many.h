// Many independent patterns on one interferometer, scheduled statically: the
// host cuts every pattern's time-state range into chunks, one wavefront per
// chunk (no shared counters), each chunk writes its own partial slot, and a
// second kernel adds every pattern's slots in slot order.
//
// Forward mode: the slot holds the chunk's double-double sum of
//   w * prod_j c_j^{kap_j}.
// Adjoint mode (reverse of the Gray-code sweep): the slot holds the chunk's
// part of D_ij = sum_states w * delta_i * G_j with G_j = d/dc_j prod_l c_l^{kap_l},
// so that d perm / d B_ij = 2^{-(n-1)} D_ij, plus the forward sum.  Per lane,
// P_j = running sum of w G_j; a step that moves digit k by dd changes delta_k
// by -2 dd, and summation by parts gives
//   sum_t delta_k(t) g(t) = delta_k(end) P(end) + sum_flips 2 dd P(before flip).
// Only the lowest KA time digits may change inside a chunk (chunks are aligned
// to their period); every other row's delta is constant over the chunk, so its
// share is delta_i * P(end), contracted over the lanes once per chunk.
#pragma once
#include <stdint.h>

#include "batch.h"
#include "pq_common.h"

namespace pq {

constexpr int kModeFwd = 0;       // forward sums (PERM jobs)
constexpr int kModeExt = 1;       // Laplace expansion along a new row (EXTEND_ROW jobs)
constexpr int kModeAdj = 2;       // reverse sweep: derivatives and forward sums
constexpr int kModeAdjWalk = 3;   // reverse sweep of wide collision-free patterns (k_adjw_impl.h)
constexpr int kModeExtCol = 4;    // EXTEND_ROW jobs over the signs of unit columns (k_extcol_impl.h)
constexpr int kExtColDigits = 8;  // most time digits that move inside one of its chunks
// Under pq_perm_batched its chunks are handed out by the dispatcher as in the
// static schedule, longest first, which evens out the CUs as a queue would: popped
// from one counter, 1000 runs of 20 photons in 400 modes take 5.7 ms instead of
// 4.5 and 100 runs 1.68 instead of 0.88 (a chunk is a quarter of a row chunk's
// work).  What a queue has besides is the host's request to stop: of the chunks
// behind the first kExtColPollFrom per CU, which start at once, every
// kExtColPollEvery-th reads the host's word and passes it on through a word in
// device memory, which the others read (with every chunk reading over the host
// link 400 jobs of 24 columns took 19.2 ms instead of 17.7, and as long when
// cancelled).
constexpr int kExtColPollFrom = 16;
constexpr int kExtColPollEvery = 64;
constexpr int kWalkMinCols = 16;  // padded column range of the walk classes
constexpr int kWalkMaxCols = 32;
constexpr int kWalkLaneStates = 16;   // lane-digit states per wavefront (four lanes per term)
constexpr int kWalkTerms = 16;        // terms per wavefront
constexpr int kWalkWaves = 4;         // wavefronts per workgroup, all on one pattern
constexpr int kManyMaxAdjCols = 24;   // widest adjoint class
constexpr int kAdjBlock = 64;         // one wavefront per workgroup in adjoint mode

struct MChunk {
    int32_t pat;          // pattern (index into the job array)
    int32_t slot;         // partial slot
    uint64_t start;
    uint64_t count;
};

struct ManyArgs {
    const BJob* jobs;       // per pattern (BJob layout; out_offset = pattern index)
    const MChunk* chunks;   // this class's chunks
    int32_t nchunks;
    int32_t slot_doubles;   // doubles per slot
    const cplx* mat;
    const int32_t* idx;
    const StepEntry* tabs;
    double* partials;       // slot storage of this class
    // kModeExtCol under pq_perm_batched: the first chunk that reads the words, the
    // host's word (pq_cancel; null: none reads) and the class's word in device
    // memory that is set from it.  (In this order: with a pointer right behind
    // partials both are loaded at once and held through the sweep, 0.5 % of
    // 1000 runs of 20 photons)
    int64_t poll_from;
    const int32_t* cancel;
    unsigned* stop;
};

// Reduction of the reverse sweeps' derivative slots in two fixed-order
// stages: stage 1 (in the final kernel) adds up to 64 consecutive slots of a
// pattern for 64 consecutive entries, stage 2 adds a pattern's stage-1 partials
// and scales; a pattern of one stage-1 row needs no second stage.
// Item (pat, eb, cb): entries [64 eb, 64 eb + 64), slots [64 cb, 64 cb + 64);
// stage-2 items have cb = 0 and read ncb partial rows.
struct DRedItem {
    int32_t pat, eb, cb, ncb;
    int64_t part_off;       // complex offset of the pattern's [ncb][r * nc] partials
};

struct DRedArgs {
    const DRedItem* items;
    const BJob* jobs;
    const int64_t* dpat_off;
    const cplx* part;
    cplx* dpat;
};

// Per-pattern reduction of the chunk slots.
struct ManyFinalArgs {
    const cplx* U;
    int64_t ldu;
    const cplx* UT;            // columns of U, transposed, or null (extend-row jobs)
    const int32_t* ut_at;      // [m]: a column's row in it
    int32_t m;
    const cplx* mat;
    const int32_t* idx;
    const int64_t* dpat_off;   // [npat]: complex offset of the pattern's D block
    const BJob* jobs;
    const int32_t* pat_slot;   // [npat]: first slot (in the class's slot array) of every pattern
    const int32_t* pat_class;  // [npat]: class index, -1 for trivial patterns
    const int64_t* class_off;  // [nclass]: double offset of the class's slots
    const int32_t* class_sd;   // [nclass]: slot doubles of the class
    const double* partials;
    const cplx* trivial;       // [npat]: value of trivial patterns
    // copies of every distinct pattern (identical op, rows and columns are
    // swept once): copy q of pattern p is dup_off[p] <= q < dup_off[p+1], with
    // its original index dup_pat[q] and output offset dup_out[q]
    const int32_t* dup_off;    // [npat + 1]
    const int32_t* dup_pat;
    const int64_t* dup_out;
    int32_t npat;              // distinct patterns
    int32_t adjoint;
    int32_t fuse_dred;         // adjoint: most chunks of a pattern whose slots its own workgroup adds
    cplx* perm;                // may be null (forward values)
    cplx* amp;                 // may be null
    cplx* dpat;                // adjoint: per pattern r x nc complex d perm / d B (scaled)
    const cplx* gperm;         // adjoint: the caller's per-copy cotangents
    cplx* gsum;                // adjoint: per distinct pattern, the sum of its copies' cotangents
    const DRedItem* red;       // [nred]: stage-1 items of the other patterns
    int32_t nred;
    cplx* red_part;
};

// Columns of U, transposed, for the extend-row jobs' final step: its lanes are
// consecutive output modes, whose entries of one column are a row of the transpose
// (in U itself every lane reads another line).
struct TransposeArgs {
    const cplx* U;
    int64_t ldu;
    int32_t m, n;
    const int32_t* col;     // [n]
    cplx* UT;               // [n][m]
};

// Persistent work queue over one class's chunks (forward and extend-row
// classes): a grid of resident wavefronts, each popping chunk indices from
// `counter` until they run out and writing each chunk's slot; the final
// kernel then adds every pattern's slots in slot order, as after the static
// schedule.  counter starts at zero (queue_prep_kernel).
struct QueueArgs {
    ManyArgs m;
    unsigned* counter;         // this class's next-chunk counter
    const int32_t* cancel;     // host-mapped word: nonzero stops the queue (pq_cancel); may be null
};

// Reset of the queue counters before the class queues run.
struct QueuePrepArgs {
    unsigned* zero;
    int32_t nzero;
};

// Scatter of the per-pattern derivatives into dU (conjugate-Wirtinger VJP).
// For every entry e = a*m + b of dU, items[offsets[e] .. offsets[e+1]) list
// the (distinct pattern, index into dpat) pairs that touch it, in pattern
// order; gperm holds each distinct pattern's summed cotangent.
struct GradScatterArgs {
    const int32_t* offsets;    // [m*m + 1]
    const int32_t* items;      // [2 * total]: pattern, then the D index (complex)
    const cplx* dpat;
    const cplx* gperm;
    int32_t m;
    cplx* dU;
    int64_t lddu;
};

}  // namespace pq
