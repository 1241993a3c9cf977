// Internal state of a libvrm context and the kernel launchers shared by the
// translation units.  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vrm.h"
#include "vrm_mlp.h"

namespace vrm {

// The device counters live in kCounterStripes copies, one per 256-byte line.
// Accumulating kernels add to the copy of their workgroup, so that the waves of
// a large launch do not queue on one address; vrm_read_counters sums the
// copies.  Fields that are assigned (not accumulated) live in copy 0.
constexpr int kCounterStripes = 64;
constexpr size_t kCounterStride = (sizeof(vrm_counters) + 255) / 256 * 256;

// Append `want` entries per thread to a queue whose tail is *counter: positions
// follow the thread order of the workgroup, with one atomic per workgroup (a
// large launch then does not queue on one address).  Every thread of the
// workgroup must call it; s_tmp is __shared__ int[17].
__device__ __forceinline__ int block_append_n(int* counter, int want, int* s_tmp)
{
    const int lane = __lane_id(), w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    int incl = want;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) s_tmp[w] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int k = 0; k < nw; ++k) {
            const int c = s_tmp[k];
            s_tmp[k] = tot;
            tot += c;
        }
        s_tmp[16] = tot ? atomicAdd(counter, tot) : 0;
    }
    __syncthreads();
    const int pos = s_tmp[16] + s_tmp[w] + incl - want;
    __syncthreads();
    return pos;
}

__device__ __forceinline__ vrm_counters* counter_stripe(vrm_counters* base)
{
    return reinterpret_cast<vrm_counters*>(reinterpret_cast<char*>(base) +
                                           (size_t)(blockIdx.x % kCounterStripes) * kCounterStride);
}

// Grid of square cells over the bounding box of the cloud (device side).
struct GridState {
    float x0, y0, cs, inv_cs;
    int32_t nx, ny, ncells, clamped;
    // kBadPos: a position the last cell build read was not finite; kBadGamma: a
    // circulation the last selection or stage-0 copy read was not finite.  While
    // either bit is set no cell index is formed and no kernel changes the cloud.
    int32_t bad;
    // bits of max |Gamma^n| (stage 0): scale of the fixed-point accumulation
    uint32_t gmax_bits;
};
// Scratch of a cell build; `done` and `bad_seen` are zero between builds.
constexpr int kBoxBlocks = 1024;
constexpr int kCellParts = 128;   // a power of two
constexpr int kPackTiles = 16384; // of 4096 particles
struct CellScratch {
    uint32_t box[4][kBoxBlocks];   // the workgroups' boxes: ordered keys of min x, min y, max x, max y
    uint64_t part[kCellParts];     // launch number over the sum of a chunk's counts
    uint64_t pack[kPackTiles];     // removal: call number, kind and count of a tile
    uint32_t ticket;
    int32_t pack_ticket;           // zero between calls
    int32_t bad_seen;
    int32_t done[17];
};

// State of a velocity sum by boxes (box, done and bad_seen as in CellScratch).
struct BoxState {
    GridState g;            // boxes as cells: x0, y0, side cs, nx x ny
    unsigned long long all_pairs;
    alignas(128) unsigned long long work;   // of the boxes, in pairs (lines of their own: atomics)
    alignas(128) unsigned long long fullest;   // particles of the fullest box over its index
    alignas(128) int32_t items;             // work items
    int32_t bad_seen;
    int32_t done[17];
    uint32_t box[4][kBoxBlocks];
};
constexpr int32_t kBadPos = 1;
constexpr int32_t kBadGamma = 2;

constexpr int kRmRounds = 8;   // rounds of an insertion's or removal's choice per wait

// Shu-Osher SSP-RK3: y_s = a y^n + b (y_(s-1) + dt f(y_(s-1))).
constexpr float kStageA[3] = {0.0f, 0.75f, 1.0f / 3.0f};
constexpr float kStageB[3] = {1.0f, 0.25f, 2.0f / 3.0f};
__device__ __forceinline__ float combined_gamma(float a, float b, float dt, float dg, float g, float g0)
{
    const float s = b * __builtin_fmaf(dt, dg, g);
    return a != 0.0f ? __builtin_fmaf(a, g0, s) : s;
}

// p[i] by a 32-bit byte offset from the (uniform) base: fewer address instructions than
// a 64-bit one per lane; indices of slots and particles are below 2^26
__device__ __forceinline__ float load32(const float* __restrict__ p, int i)
{
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p) + 4u * (uint32_t)i);
}

// Queue counters of a stage (device side).
struct Queues {
    int32_t n_small;       // items in the small-LP queue
    int32_t n_full;        // items in the complete-LP queue
    int32_t n_cand;        // insertion candidates
    int32_t n_accepted;    // accepted insertion candidates
    int32_t small_state;   // insertion: 0 many candidates, 1 done by one workgroup, 2 capacity exceeded,
                           // 3 done in rounds, 4 chosen in rounds, keys to be sorted
    int32_t n_retry;       // LPs left by the warm pass for a cold solve
    int32_t blocks_done;   // blocks of the last LP launch that have finished
    int32_t last_small;    // n_small and n_full of the last stencil run (the queues
    int32_t last_full;     // themselves are zero between runs)
    int32_t n_rm_uncertified;   // particle removal: particles whose optimality was not certified
    int32_t rm_open[8];    // round k of a batch (insertion, removal) left candidates undecided
    int32_t nonfinite;     // copy of GridState::bad taken when the record is published
    int32_t n_defer;       // complete LPs whose certification was deferred to a second launch
    int32_t n_now;         // the cloud's count when the record was published
    int32_t done_part[16]; // blocks_done of every sixteenth block (last_block)
};

// True in one thread of the last workgroup of a launch to get here (call it with one
// thread of each, after the workgroup's last read of the counters that the last one
// will reset).  Two levels: 1280 workgroups on one address took 23 us to count.
__device__ __forceinline__ bool last_block(Queues* qs)
{
    const int part = blockIdx.x & 15, in_part = ((int)gridDim.x - part + 15) / 16;
    if (atomicAdd(&qs->done_part[part], 1) != in_part - 1) return false;
    qs->done_part[part] = 0;
    if (atomicAdd(&qs->blocks_done, 1) != min((int)gridDim.x, 16) - 1) return false;
    qs->blocks_done = 0;
    return true;
}

// True in every thread of the last workgroup to get here; what the others wrote with
// atomics whose results they waited for is complete then.  Two levels, so that the
// workgroups do not queue on one address (18 ns each); done[17] is left zero.
__device__ __forceinline__ bool last_here(int32_t* done)
{
    __shared__ int s_last;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int part = blockIdx.x & 15, in_part = ((int)gridDim.x - part + 15) / 16;
        bool last = atomicAdd(&done[part], 1) == in_part - 1;
        if (last) last = atomicAdd(&done[16], 1) == min((int)gridDim.x, 16) - 1;
        s_last = last;
    }
    __syncthreads();
    if (s_last && threadIdx.x < 17) done[threadIdx.x] = 0;
    return s_last != 0;
}

// Queue record published to pinned, coherent host memory: the kernel writes q,
// then seq last with a system-scope release; the host reads q once it sees the
// sequence number it asked for.
struct HostQueues {
    Queues q;
    int32_t seq;
};

// One thread copies the queue record (and the cloud's count) to the host copy, then
// writes the sequence number with a system-scope release (after a system fence).
__device__ __forceinline__ void publish(const Queues* q, const GridState* g, int n_now, HostQueues* h, int32_t seq)
{
    if (q) {
        h->q = *q;
        h->q.nonfinite = g->bad;
    }
    h->q.n_now = n_now;
    __threadfence_system();
    __hip_atomic_store(&h->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}


// Column records of the queued small-neighbourhood LPs, in queue order and
// plane-major (plane p of item r at p * cap + r) so that the LP and network
// kernels read them coalesced instead of gathering neighbours.
struct SmallRec {
    int32_t cap;     // plane stride
    int32_t* i;      // [cap] cloud index of the particle
    int32_t* rank;   // [cap] id ranks of its 8 columns, 3 bits each (segment s at bit 3 s)
    int32_t* pj;     // [8][cap] cloud index of the column of segment s, -1 if the segment is empty
    float* off;      // [32][cap] exact scaled offset of segment s: planes 4s..4s+3 = X.hi, X.lo, Y.hi, Y.lo
};

// Column records of the queued complete LPs, as the network's inference reads them.
struct FullRec {
    const int32_t* rec;      // [item][row] (slot << 6) | id rank per column, nearest first
    int32_t row;             // record row stride
    const int32_t* kcol;     // [item] column count; -1: the list is left for the run's last launch
    const int32_t* q_full;   // [item] sorted-cloud index of the particle
    const float* xs;         // sorted positions
    const float* ys;
    float scale2e, sc;       // ((x_j - x_i) scale2e) sc is column j's offset over h
    int q;
};

// Reduced-operator selection state (device side).
struct SelectState {
    double norm1, bound, prefix;
    uint32_t key_prefix;   // resolved high bits of the threshold key
    uint32_t done;         // 1 once the threshold is known
    uint32_t threshold;    // particles with key < threshold are left out
    int32_t max_id;        // largest id of the cloud (new particles get max_id + 1, ...)
    uint32_t max_seen;     // of the first pass, zero between selections: largest id + 1,
    int32_t bad_seen;      // a non-finite circulation,
    int32_t done_blocks[17];   // finished workgroups of a pass
};
constexpr int kSelBins = 2048;   // bins of a context's radix passes (11, 11 and 10 bits)

struct LaunchParams {
    float h, lo2, hi2, lo2f, hi2f;      // annulus bounds (FP32, squared, unnormalised)
    float rad, ex2;                      // insertion radius 1.5 h and exclusion (0.5 h)^2
    float scale2e;                       // 2^-e with 2^e >= h: exact offset scaling
    float bt_hi, bt_lo;                  // rhs 2 h^2 / 4^e of the (2,0), (0,2) rows (double-float)
    float cs_hi, cs_lo;                  // (2^e / h)^(q+1): cost scale (double-float)
    float lam;                           // nu / h^2
    float sc;                            // 2^e / h: scaled offset -> offset / h
    int q, m;
    int phase1;                          // 1: stop at the first feasible vertex (phase I only)
    int det;                             // 1: order-independent fixed-point accumulation of the update
    int max_cert;                        // certification rounds of one LP (kMaxCert unless tuned)
};
constexpr int kMaxCert = 8;              // certification rounds: primal / dual repairs of one LP
// A kept stencil: a row of 12 column indices and one of 12 fractions (48 bytes
// each: three 16-byte accesses).  At most nine columns carry a fraction; the
// last index holds their count, or -1 for a particle without a stencil, and the
// last fraction fhat_ii.
constexpr int kStenRow = 12;
// what a stencil run leaves in the kept rows: nothing; the stencils; the columns that
// carry the fractions (the basis from which a later stage's LPs start)
constexpr int kKeepNone = 0, kKeepStencils = 1, kKeepBases = 2;

// Fixed-point accumulation (deterministic mode): every contribution f Gamma is
// rounded to a multiple of 2^(e - 46), where max |Gamma^n| < 2^e, and summed as
// a 64-bit integer, so the sum does not depend on the order of the atomics and
// particles with equal contributions get bit-identical sums.  A fraction is at
// most 16 (Sec. 3.2 lemma: sum_{j != i} fhat_ij <= 4 / r^2), a stage value at
// most 4 max|Gamma^n|, and a particle receives at most 2^10 contributions, so
// every scaled sum stays below 2^62 in magnitude.
__device__ __forceinline__ double det_scale(uint32_t gmax_bits)
{
    const int e = (int)((gmax_bits >> 23) & 255u) - 126;   // max|Gamma| < 2^e
    return __builtin_ldexp(1.0, 46 - e);
}
__device__ __forceinline__ void acc_add(float* acc, int j, float f, float g, double dsc)
{
    if (dsc != 0.0)
        atomicAdd(reinterpret_cast<unsigned long long*>(acc) + j,
                  (unsigned long long)(long long)__builtin_rint((double)f * (double)g * dsc));
    else
        atomicAdd(acc + j, f * g);
}

// The kept rows of a context, by particle index: [cap][kStenRow] columns, then
// [cap][kStenRow] fractions, in scratch that the runs of their order do not use (the
// column lists of the nine-row LPs, the column records of the five-row ones).
struct StenRows {
    int32_t* idx;
    float* f;
};

// A context's small device state that starts as zero: one allocation and one clear (a small
// context took 140 us to create with one of each for every part, now 76).
struct FixedState {
    alignas(256) GridState grid;
    alignas(256) Queues queues;
    alignas(256) SelectState sel;
    alignas(256) double sel_bins[kSelBins];
    alignas(256) char counters[kCounterStripes * kCounterStride];
    alignas(256) CellScratch cell_scratch;
    alignas(256) BoxState bs_state;
    alignas(256) int32_t khist[2 * (VRM_KMAX + 1)];
};

}  // namespace vrm

struct vrm_ctx {
    int device;
    hipStream_t stream;
    int32_t capacity;
    int32_t ncell_cap;
    // cached count for the cloud last seen (host)
    const int32_t* n_ptr;
    int32_t n;
    int32_t n_diffused_valid;   // the diffused set matches the cloud
    int32_t cells_valid;        // cell list matches the current positions
    int32_t base_valid;         // y^n recorded (stage 0 done)
    int32_t sorted;             // cloud in cell order of the current cell list (perm is the identity)
    const float* cloud_x;       // cloud seen last (cached state belongs to it)
    float* u_tmp;               // [cap] stage velocity (vrm_step with prescribed vortices)
    float* v_tmp;
    // device buffers
    vrm::FixedState* fixed;     // holds grid, queues, sel, sel_bins, counters, cell_scratch, bs_state, khist
    vrm::GridState* grid;
    vrm::Queues* queues;
    vrm::HostQueues* q_host;    // pinned, coherent host copy of *queues (vrm_read_queues)
    int32_t q_seq;              // last sequence number asked of it
    vrm::SelectState* sel;
    double* sel_bins;     // [kSelBins] sums of a radix pass, zero between selections
    vrm_counters* counters;
    int32_t* cell_count;  // [ncell_cap + 8] particles per cell, zero between builds
    int32_t* rank;        // [cap] rank within its cell
    int32_t* cell_start;  // [ncell_cap + 1]
    vrm::CellScratch* cell_scratch;
    vrm::BoxState* bs_state;
    int32_t* perm;        // [cap] slot -> particle
    float* xs;            // [cap] positions in slot order
    float* ys;
    int32_t* ids;         // [cap] ids in slot order
    uint8_t* diffused;    // [cap] per particle
    float* acc;           // [2 cap] sum_j fhat_ji Gamma_j (FP32, or int64 fixed point when deterministic)
    float* x0;            // [cap] stage-0 state
    float* y0;
    float* g0;
    int32_t* q_small;     // [cap] slots queued for the small LP
    int32_t* q_full;      // [cap] slots queued for the complete LP
    int32_t* q_retry;     // [cap] slots the warm pass leaves for a cold solve
    vrm::SmallRec srec;   // column records of the queued small LPs
    // insertion
    float* cx;            // [2 cap] candidate positions
    float* cy;
    uint64_t* ckey;       // [2 cap] (id << 3) | segment
    uint8_t* cstate;      // [2 cap] 0 undecided, 1 in, 2 out
    int32_t* crank;
    int32_t* cstart;      // [ncell_cap + 1]
    int32_t* cperm;       // [2 cap]
    uint64_t* akey;       // [2 cap] accepted keys / sort scratch
    int32_t* aidx;
    void* sort_tmp;
    size_t sort_tmp_bytes;
    // reorder scratch
    float* tmp_f;         // [3 cap]
    int32_t* tmp_i;       // [cap]
    uint8_t* tmp_u8;      // [cap]
    int lp_objective;     // 0 canonical stencil (phase II), 1 first feasible vertex (phase I only)
    // kernel timers
    int timing;
    uint32_t timing_groups;   // bit g: group g is timed
    int ntimed;
    hipEvent_t* ev_start; // [kMaxTimed]
    hipEvent_t* ev_stop;
    int* ev_group;
    int64_t launches[VRM_NTIMER];
    double acc_ms[VRM_NTIMER];   // timings accumulated from graph replays
    int64_t acc_n[VRM_NTIMER];
    // the three stages of vrm_step as one HIP graph
    int capturing;               // the stream is being captured: timers take graph slots
    int graph_enabled;
    int64_t graph_replays;
    int graph_failed[2];         // capture failed (without / with timers): launch directly
    int graph_slots;             // timer slots used by the graph
    int graph_pending;           // a replay whose timer events are not yet accumulated
    int graph_nb;                // particle bound the graph's grids are sized for
    int graph_flags[3];          // cells_valid, sorted, base_valid after the stages
    hipGraph_t graph;
    hipGraphExec_t graph_exec;
    unsigned char graph_key[256];
    double* t_dev;               // step start time read by the graph's velocity kernels
    int32_t* prev;               // [cap][9] basis (column ids) of each particle's last stencil, by id
    uint64_t* pmask;             // [cap] crash basis (previous or predicted) as a column mask per complete LP
    int32_t* lkey;               // [cap] bin of each complete LP for the counting sort (pivot history or doubt)
    int32_t* q_defer;            // [cap] queue items the LP launch deferred (bit 31: settled warm; bit 30: solve cold)
    uint8_t* pivhist;            // [cap] by particle id: pivots of its last complete LP (255: none yet)
    vrm_tuning tuning;           // launch shapes in force (defaults filled in)
    hipStream_t cap_stream;      // stream the graph is captured on (the context's may be the null stream)
    // warm-start network (allocated on first use)
    vrm::MlpState* mlp;
    int warm;             // LP solves use the network's basis prediction
    uint16_t* feat;       // [cap][128] feature rows of the queued LPs (warm start / collection)
    float* pred;          // [cap][64] network outputs
    float* labels;        // [cap][64] collection targets
    int32_t* full_cols;   // [cap][48] complete-neighbourhood columns nearest first: (slot << 6) | id rank
    int32_t* full_k;      // [cap] their counts, by queue item
    int32_t* full_order;  // [cap] queue items grouped by decreasing count
    int32_t* khist;       // [2 (VRM_KMAX + 1)] histogram of the counts, then the bins' fill pointers
    int32_t feat_cap;
};

namespace vrm {
inline StenRows sten_rows(const vrm_ctx* c, int m)
{
    static_assert(2 * kStenRow <= VRM_KMAX && 2 * kStenRow <= 4 * VRM_NSEG, "the rows fit in the scratch");
    int32_t* p = m == 5 ? c->full_cols : reinterpret_cast<int32_t*>(c->srec.off);
    return {p, reinterpret_cast<float*>(p + (size_t)c->capacity * kStenRow)};
}
constexpr int kMaxTimed = 8192;
constexpr int kGraphTimed = 64;   // the last kGraphTimed event pairs belong to the step graph
// Bracket a group of launches with events when timing is on.
struct ScopedTimer {
    vrm_ctx* c;
    int slot;
    ScopedTimer(vrm_ctx* ctx, int group) : c(ctx), slot(-1)
    {
        if (!c->timing || !((c->timing_groups >> group) & 1u)) return;
        if (c->capturing) {
            // an event-record node of the step graph; counted when a replay is accumulated
            if (c->graph_slots >= kGraphTimed) return;
            slot = kMaxTimed - kGraphTimed + c->graph_slots++;
        } else {
            c->launches[group] += 1;
            if (c->ntimed >= kMaxTimed - kGraphTimed) return;
            slot = c->ntimed++;
        }
        c->ev_group[slot] = group;
        (void)hipEventRecord(c->ev_start[slot], c->stream);
    }
    ~ScopedTimer()
    {
        if (slot >= 0) (void)hipEventRecord(c->ev_stop[slot], c->stream);
    }
};
}  // namespace vrm

// launchers (vrm_cells.hip)
int vrm_build_cells(vrm_ctx* c, const float* x, const float* y, const int32_t* id, int32_t n,
                    const vrm::LaunchParams& lp, const int32_t* n_dev = nullptr);
int vrm_select_run(vrm_ctx* c, const vrm_cloud* cl, int32_t guess, double bound_factor, int32_t& n);
int vrm_cell_slots(vrm_ctx* c, const vrm::GridState* g, const float* x, const float* y, int32_t n,
                   const int32_t* n_dev, int32_t* start, int32_t* rank);
int vrm_select_mask_run(vrm_ctx* c, const float* gamma, int32_t n, uint8_t* mask_out);
int vrm_select_init(vrm_ctx* c);
int vrm_insert_run(vrm_ctx* c, vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp);
// the queue record after the work enqueued so far on the context's stream,
// read from the pinned host copy (no stream synchronisation); n_now of n_dev unless NULL
int vrm_read_queues(vrm_ctx* c, vrm::Queues& q, const int32_t* n_dev = nullptr);
// the record a kernel publishes with the number seq
int vrm_wait_queues(vrm_ctx* c, int32_t seq, vrm::Queues& q);
int vrm_reorder_cloud(vrm_ctx* c, vrm_cloud* cl, int32_t n);
int vrm_remove_run(vrm_ctx* c, vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp, bool stored,
                   int32_t* n_candidates);
// launchers (vrm_lp.hip)
int vrm_stencil_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp,
                    const vrm_stencils* out, int apply, uint16_t* feat_out = nullptr, float* label_out = nullptr,
                    int max_rows = 0, int keep = vrm::kKeepNone, bool from_bases = false);
// the update of the stencils kept by a vrm_stencil_run with kKeepStencils
int vrm_combine_apply_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp, int stage, double dt,
                          int half);
int vrm_apply_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp);
int vrm_small_nbhd_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp,
                       int32_t* small_idx, int32_t* kfull);
int vrm_warm_predict_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp, float* out,
                         int32_t* particle, int max_rows);
// launchers (vrm_stage.hip)
int vrm_combine_run(vrm_ctx* c, vrm_cloud* cl, int32_t n, const float* u, const float* v, double dt,
                    float lam, int stage, int det);
int vrm_save_base_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, int det);
int vrm_biot_savart_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, double eps, float* u, float* v);
int vrm_verify_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const vrm::LaunchParams& lp, double h,
                   const vrm_stencils* st, double* report);
int vrm_velocity_run(vrm_ctx* c, const vrm_cloud* cl, int32_t n, const float* vort, int32_t nv, double nu,
                     double t, float* u, float* v, const double* t_dev = nullptr);

// launchers (vrm_mlp.hip)
int vrm_mlp_alloc(vrm_ctx* c, int max_rows);
void vrm_mlp_free(vrm_ctx* c);
int vrm_mlp_set_weights(vrm_ctx* c, const float* w_dev);
int vrm_mlp_read_weights(vrm_ctx* c, float* w_dev);
int vrm_mlp_infer_run(vrm_ctx* c, const uint16_t* X, int rows, float* Y, const int* rows_dev);
// warm-start logits (8 per queued small LP) with the network input built from the positions
int vrm_mlp_infer_full_run(vrm_ctx* c, int rows, const int* rows_dev, const vrm::FullRec& fr, float* L);
int vrm_mlp_infer_small_run(vrm_ctx* c, int rows, const int* rows_dev, const vrm::SmallRec& rec, float sc, int q,
                            float* L);
int vrm_mlp_train(vrm_ctx* c, const uint16_t* X, const float* T, int rows, float lr, float wd, float wf,
                  double* loss_out, float* grad_out);
int vrm_gemm_test(vrm_ctx* c, const uint16_t* A, const uint16_t* B, float* C, int M, int N, int K, int transA,
                  int transB);

// error helpers (vrm_api.cpp)
int vrm_fail(int code, const char* fmt, ...);
// report a non-finite input (GridState::bad bits): clears the device flag and
// drops the context's cached cell list and diffused set; returns VRM_E_NONFINITE
int vrm_nonfinite(vrm_ctx* c, int32_t bits);
int vrm_hip_check(hipError_t e, const char* what);
#define VRM_HIP(call)                                                    \
    do {                                                                 \
        hipError_t _e = (call);                                          \
        if (_e != hipSuccess) return vrm_hip_check(_e, #call);           \
    } while (0)
