// C ABI of libkge: argument checks, workspace, and the order in which the kernels of one step are enqueued.
// See include/kge.h for the contract of each entry point.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>
#include <new>

#include "kge_common.h"
#include "k_weights.h"

// Scratch memory of kge_score_noalloc, the one entry point that allocates nothing: a fixed array in the library's
// device image (every GPU that runs the library holds its own copy until the process ends).  In host code the name
// below is only a handle for hipGetSymbolAddress; the address the kernels get is the one that call returns.
constexpr size_t KGE_NOALLOC_SCRATCH_BYTES = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[KGE_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int KGE_MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[KGE_MAX_DEVICES] = {};  // per device: where that GPU's copy of `scratch` lives

// Address of the current device's scratch array (resolved once per device, with that device current).
hipError_t scratch_address(int device, void** out) {
    if (device < 0 || device >= KGE_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

thread_local char g_create_err[512] = "";

int fail(kge_ctx* c, int code, const char* fmt, const char* detail = "") {
    char* dst = c ? c->err : g_create_err;
    snprintf(dst, 512, fmt, detail);
    return code;
}

#define KGE_HIP(c, call)                                                                 \
    do {                                                                                 \
        hipError_t e_ = (call);                                                          \
        if (e_ != hipSuccess) return fail((c), KGE_ERR_DEVICE, #call ": %s", hipGetErrorString(e_)); \
    } while (0)

bool is_gemm_model(int m) { return m == KGE_TRANSE_L2 || m == KGE_DISTMULT || m == KGE_COMPLEX || m == KGE_RESCAL; }

__global__ void k_validate(StepIds ids, int64_t n_ent, int64_t n_rel, int* flag) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const StepView v = step_view(ids);
    bool bad = false;
    if (i < ids.b)
        bad = v.h[i] < 0 || v.h[i] >= n_ent || v.t[i] < 0 || v.t[i] >= n_ent || v.r[i] < 0 || v.r[i] >= n_rel;
    if (i < ids.n_neg) bad = bad || v.neg[i] < 0 || v.neg[i] >= n_ent;
    if (bad) atomicOr(flag, 1);
}

void launch_validate(kge_ctx* c, const StepIds& ids, hipStream_t st) {
    const int n = ids.b > ids.n_neg ? ids.b : ids.n_neg;
    hipLaunchKernelGGL(k_validate, dim3((n + 255) / 256), dim3(256), 0, st, ids, c->cfg.num_entities,
                       c->cfg.num_relations, c->flags);
}

StepIds direct_ids(const int64_t* h, const int64_t* r, const int64_t* t, int b, const int64_t* neg, int n_neg, int side,
                   float* loss_out) {
    StepIds ids;
    ids.h = h; ids.r = r; ids.t = t; ids.neg = neg; ids.b = b; ids.n_neg = n_neg; ids.side = side;
    ids.blk = nullptr; ids.loss_out = loss_out;
    return ids;
}

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

int check_batch(kge_ctx* c, const void* ent, const void* rel, const int64_t* h, const int64_t* r, const int64_t* t,
                int64_t b, const int64_t* neg, int64_t k, int64_t chunk, int32_t side, bool need_neg) {
    if (!ent || !rel || !h || !r || !t) return fail(c, KGE_ERR_INVALID_ARG, "null table or id pointer%s");
    if (b <= 0 || chunk <= 0 || b % chunk != 0) return fail(c, KGE_ERR_INVALID_ARG, "b must be a positive multiple of chunk%s");
    if (k < 0 || (need_neg && k == 0)) return fail(c, KGE_ERR_INVALID_ARG, "k out of range%s");
    if (k > 0 && !neg) return fail(c, KGE_ERR_INVALID_ARG, "neg is null%s");
    if (side != KGE_NEG_TAIL && side != KGE_NEG_HEAD) return fail(c, KGE_ERR_INVALID_ARG, "neg_side must be 0 or 1%s");
    if (b > c->cfg.max_batch || k > c->cfg.max_neg_per_chunk || b / chunk > c->cfg.max_chunks)
        return fail(c, KGE_ERR_WORKSPACE, "b, k or b/chunk exceed the sizes given to kge_create%s");
    return KGE_OK;
}

void forward(kge_ctx* c, const float* ent, const float* rel, const StepIds& ids, int k, int chunk, float gamma,
             float* pos_out, float* neg_out, int ld_out, int dist_mode, hipStream_t st) {
    if (c->cfg.validate_indices) launch_validate(c, ids, st);
    if (kge_ind_score_fits(c, chunk)) {
        kge_ind_score(c, ent, rel, ids, k, gamma, k > 0 ? neg_out : nullptr, ld_out, pos_out, st);
        return;
    }
    if (c->cfg.model == KGE_RESCAL) kge_launch_rescal_phi(c, ent, rel, ids, st);
    // (TransE-L1's sums have the same order there.  The others' have not, and ranks of candidates that tie with the positive hang
    // on the last bit: see split_forward in k_gemm.hip)
    if (c->cfg.model == KGE_TRANSE_L1 && neg_out && k > 0 && dist_mode == 0 && kge_front_fits(c, ids.b, k, chunk, false)) {
        kge_launch_front(c, ent, rel, ids, k, chunk, gamma, pos_out, false, false, neg_out, ld_out, dist_mode, st);
        return;
    }
    kge_launch_gather(c, ent, rel, ids, chunk, gamma, pos_out, false, st);
    if (c->cfg.model == KGE_TRANSR) kge_transr_phi(c, ent, rel, ids, chunk, gamma, pos_out, false, false, st);
    if (neg_out && k > 0) {
        if (c->cfg.model == KGE_TRANSR) {
            kge_transr_project(c, rel, ids, k, chunk, gamma, neg_out, ld_out, false, false, st);
        } else if (is_gemm_model(c->cfg.model)) {
            kge_gemm_neg_score(c, ids.b, k, chunk, gamma, neg_out, ld_out, dist_mode, st);
        } else {
            kge_pair_neg_score(c, ids.b, k, chunk, gamma, neg_out, ld_out, st);
        }
    }
}

// ---- optional per-kernel timing (kge_profile): the one kernel launched inside a scope carries the scope's two
// events as its start / stop events (KGE_LAUNCH), the stream is synchronised after the step, and the elapsed times
// of the scopes that launched something are accumulated per slot.  (Events that no launch has carried cannot be read, those of an
// earlier step's launch would be counted again.)
struct ProfScope {
    kge_ctx* c;
    int slot;
    ProfScope(kge_ctx* c_, int slot_) : c(c_), slot(slot_) {
        if (c->prof_on) { c->launch_ev0 = c->prof_ev[slot][0]; c->launch_ev1 = c->prof_ev[slot][1]; }
    }
    ~ProfScope() {
        if (c->prof_on && !c->launch_ev0) c->prof_launched |= 1u << slot;
        c->launch_ev0 = nullptr; c->launch_ev1 = nullptr;
    }
};

int end_of_step(kge_ctx* c, hipStream_t st) {
    KGE_HIP(c, hipGetLastError());
    if (c->prof_on) {
        KGE_HIP(c, hipStreamSynchronize(st));
        for (int s = 0; s < KGE_PROF_SLOTS; ++s) {
            float ms = 0.f;
            if (!(c->prof_launched >> s & 1)) continue;
            if (hipEventElapsedTime(&ms, c->prof_ev[s][0], c->prof_ev[s][1]) == hipSuccess) c->prof_ms[s] += ms;
        }
        c->prof_steps += 1;
    }
    return KGE_OK;
}

// TransR after its gather launch.  Profile slots: phi, neg_score = projections and scores (in one pass with dL/dP and the
// back-projection of the corrupting rows where k_transr_project_units runs), loss, chain = dL/dP and dL/do (or what is left of
// dL/do), neg_backward = the back-projection (or nothing), rel_update, update; dL/dM is not timed.
int enqueue_transr_rest(kge_ctx* c, float* ent, float* ent_state, float* rel, float* rel_state, const StepIds& ids,
                        int K, int G, float gamma, float lr, bool beside, hipStream_t st) {
    // (rows of more than KGE_SHORT_SCORES scores: the loss kernel, with the functions it has for them)
    const bool form_w = kge_gemm_backward_forms_w(c) && K <= KGE_SHORT_SCORES;
    int n_loss_parts;
    {
        ProfScope p(c, KGE_PROF_PHI);
        kge_transr_phi(c, ent, rel, ids, G, gamma, nullptr, true, form_w, st);
    }
    {
        ProfScope p(c, KGE_PROF_SCORE);
        n_loss_parts = kge_transr_project(c, rel, ids, K, G, gamma, c->S, c->ld_s, true, form_w, st);
    }
    if (!form_w) {
        ProfScope p(c, KGE_PROF_LOSS);
        kge_launch_loss(c, ids.b, K, gamma, st);
    }
    {
        ProfScope p(c, KGE_PROF_CHAIN);
        kge_transr_dp(c, ids, K, G, form_w, st);
    }
    {
        ProfScope p(c, KGE_PROF_BACKWARD);
        kge_transr_back(c, rel, ids, K, G, form_w, st);
    }
    kge_transr_mgrad(c, ent, rel, ids, K, G, form_w, st);
    if (beside) KGE_HIP(c, hipStreamWaitEvent(st, c->ev_join, 0));
    {
        ProfScope p(c, KGE_PROF_REL_UPDATE);
        kge_transr_update(c, rel, rel_state, ids, lr, form_w, st);
    }
    {
        ProfScope p(c, KGE_PROF_UPDATE);
        kge_launch_update(c, ent, ent_state, rel, rel_state, ids, lr, n_loss_parts, true, st);
    }
    return end_of_step(c, st);
}

// Chunks of one positive.  Profile slots: gather = the key order, neg_backward = k_ind, update = the entity rows (without
// the join of runs that cross tiles), rel_update = relation rows and loss.
int enqueue_ind_rest(kge_ctx* c, float* ent, float* ent_state, float* rel, float* rel_state, const StepIds& ids, int K,
                     float gamma, float lr, bool long_lists, bool beside, hipStream_t st) {
    if (!long_lists) {
        ProfScope p(c, KGE_PROF_GATHER);
        kge_launch_key_order(c, ids, st);
    }
    {
        ProfScope p(c, KGE_PROF_BACKWARD);
        kge_ind_step(c, ent, rel, ids, K, gamma, st);
    }
    if (beside) KGE_HIP(c, hipStreamWaitEvent(st, c->ev_join, 0));
    {
        ProfScope p(c, KGE_PROF_UPDATE);
        kge_launch_update_runs(c, ent, ent_state, ids, K, lr, st);
    }
    {
        ProfScope p(c, KGE_PROF_REL_UPDATE);
        kge_launch_update(c, ent, ent_state, rel, rel_state, ids, lr, 0, false, st);
    }
    return end_of_step(c, st);
}

int enqueue_step(kge_ctx* c, float* ent, float* ent_state, float* rel, float* rel_state, const StepIds& ids, int K,
                 int G, float gamma, float lr, hipStream_t st) {
    const int B = ids.b;
    c->prof_launched = 0;
    // Ordering the key lists needs only the ids.  Short lists are ordered by extra blocks of the gather launch; long ones by a
    // radix sort, on a second stream that joins before the update.  A fork and a join cost about 10 us each outside of a graph,
    // and k_ind slows down what runs beside it, so steps of chunks of one positive that are launched one by one sort on the
    // main stream, but where k_ind (a workgroup per positive) has more workgroups than the chip holds, whose second round
    // leaves room for the sort, and work enough.  us per step, main stream / beside (b, k, D):
    //   TransE-L2  1024, 256, 400 146 / 153;  512, 128, 400 81 / 88;  1536, 256, 400 215 / 210;  2048, 512, 200 328 / 316
    //   DistMult   1024, 512, 400 262 / 269;  1280, 128, 400 117 / 121;  2048, 128, 400 148 / 156;  1280, 200, 400 152 / 150;  1280, 256,
    //              400 190 / 187;  2048, 256, 400 268 / 259;  2048, 512, 400 476 / 454;  rows of more than 512 floats, of which the chip
    //              holds half as many: 512, 256, 800 154 / 162;  1024, 128, 640 147 / 139;  1024, 256, 640 218 / 208
    //   ComplEx    1024, 256, 400 145 / 153;  1280, 256, 400 197 / 187;  2048, 512, 400 482 / 449;  1024, 256, 640 218 / 208
    //   TransE-L1  1024, 256, 400 185 / 191;  1280, 256, 400 244 / 237;  2048, 512, 400 614 / 576;  1024, 256, 640 298 / 286
    //   RotatE     (three workgroups per CU instead of four)  700, 256, 400 146 / 151;  800, 256, 400 176 / 166;  1024, 192, 400 167 /
    //              162;  1024, 256, 400 203 / 194;  1024, 200, 256 122 / 124;  2048, 128, 256 149 / 156
    // Replayed steps (TransE-L2 1024, 256, 400 147.5 beside, 148) and chunks of more positives (TransE-L2 b 2048, g 8, k 64, D 200
    // 87 beside, 92) sort beside.
    const bool long_lists = 2 * B + ids.n_neg > KGE_RANK_MAX_KEYS, ind = kge_ind_step_fits(c, G);
    const bool rotate = c->cfg.model == KGE_ROTATE, long_rows = c->cfg.ent_dim > 512;
    const bool long_ind = B > (long_rows ? 512 : rotate ? 768 : 1024) &&
                          (int64_t)ids.n_neg * c->cfg.ent_dim >= (int64_t)(rotate || long_rows ? 72 : 120) << 20;
    const bool beside = long_lists && (!ind || ids.blk || long_ind);
    if (long_lists && !beside) {
        ProfScope p(c, KGE_PROF_SORT);
        kge_launch_sort(c, ids, st);
    }
    if (beside) {
        KGE_HIP(c, hipEventRecord(c->ev_fork, st));
        KGE_HIP(c, hipStreamWaitEvent(c->side_stream, c->ev_fork, 0));
        {
            ProfScope p(c, KGE_PROF_SORT);
            kge_launch_sort(c, ids, c->side_stream);
        }
        KGE_HIP(c, hipEventRecord(c->ev_join, c->side_stream));
    }
    if (c->cfg.validate_indices) launch_validate(c, ids, st);
    if (ind) return enqueue_ind_rest(c, ent, ent_state, rel, rel_state, ids, K, gamma, lr, long_lists, beside, st);
    if (c->cfg.model == KGE_RESCAL) {
        ProfScope p(c, KGE_PROF_PHI);
        kge_launch_rescal_phi(c, ent, rel, ids, st);
    }
    const bool front = kge_front_fits(c, B, K, G, !long_lists);
    if (front) {
        ProfScope p(c, KGE_PROF_GATHER);
        kge_launch_front(c, ent, rel, ids, K, G, gamma, nullptr, true, !long_lists, c->S, c->ld_s,
                         !is_gemm_model(c->cfg.model) ? 0 : kge_gemm_backward_forms_w(c) ? 2 : 1, st);
    } else {
        ProfScope p(c, KGE_PROF_GATHER);
        kge_launch_gather(c, ent, rel, ids, G, gamma, nullptr, !long_lists, st);
    }
    if (c->cfg.model == KGE_TRANSR) return enqueue_transr_rest(c, ent, ent_state, rel, rel_state, ids, K, G, gamma, lr, beside, st);
    if (!front) {
        ProfScope p(c, KGE_PROF_SCORE);
        if (is_gemm_model(c->cfg.model))
            kge_gemm_neg_score(c, B, K, G, gamma, c->S, c->ld_s, kge_gemm_backward_forms_w(c) ? 2 : 1, st);
        else kge_pair_neg_score(c, B, K, G, gamma, c->S, c->ld_s, st);
    }
    // The matrix-product models fold the loss (uniform weights) and the chain rule (TransE-L2, DistMult) into
    // the backward launch; whatever is not folded runs as its own kernel.
    const bool gemm = is_gemm_model(c->cfg.model);
    const bool run_loss = gemm && !kge_gemm_backward_forms_w(c);
    const bool run_chain = !(gemm && kge_gemm_backward_does_chain(c));
    int n_loss_parts = gemm ? kge_gemm_loss_parts(c, B, K, G) : 0;
    if (run_loss) {
        ProfScope p(c, KGE_PROF_LOSS);
        kge_launch_loss(c, B, K, gamma, st);
    }
    {
        ProfScope p(c, KGE_PROF_BACKWARD);
        if (gemm) kge_gemm_neg_backward(c, ent, rel, ids, K, G, gamma, st);
        else n_loss_parts = kge_pair_neg_backward(c, B, K, G, gamma, st);
    }
    const bool by_runs = c->cfg.model == KGE_RESCAL && kge_rescal_chain_by_runs(c);  // the chain rule needs the relations' order
    if (beside && by_runs) KGE_HIP(c, hipStreamWaitEvent(st, c->ev_join, 0));
    if (run_chain) {
        ProfScope p(c, KGE_PROF_CHAIN);
        if (c->cfg.model == KGE_RESCAL) kge_launch_rescal_chain(c, ent, rel, ids, !beside || by_runs, st);
        else kge_launch_chain(c, ent, rel, ids, st);
    }
    if (beside && !by_runs) KGE_HIP(c, hipStreamWaitEvent(st, c->ev_join, 0));
    if (c->cfg.model == KGE_RESCAL) {
        ProfScope p(c, KGE_PROF_REL_UPDATE);
        kge_launch_rescal_update(c, ent, rel, rel_state, ids, lr, st);
    }
    {
        ProfScope p(c, KGE_PROF_UPDATE);
        kge_launch_update(c, ent, ent_state, rel, rel_state, ids, lr, n_loss_parts, true, st);
    }
    return end_of_step(c, st);
}

// ---- replay: kge_train_steps captures 16 or 32 consecutive steps into HIP graphs whose kernels take the step
// number and the id arrays from device memory (the step block), so the same graphs serve every step of every call
// of the same shape.  A graph costs the host about 0.7 us per kernel where a plain launch costs 3.7 us, and costs the
// device about 8 us of idling at its start where plain launches follow each other without a gap as long as the host
// stays ahead (it does: 15 us of launching per four-kernel step against 20 us and more on the device; and a plain
// launch carries its id pointers in its arguments, one dependent load less per kernel).  So:
//   fewer than 16 steps       plain launches
//   up to REPLAY_LONG steps   plain launches, and one graph for the last 16 or 32 steps (the call returns while they run);
//                             the first such call plain launches only
//   longer calls              plain launches for at least 32 steps, graphs of 32 for the rest
// Measured per pass (all graphs, growing from one step -> this): 4 TransE-L1 steps 223 -> 201 us, 50 RotatE steps 3940 ->
// 3890, 100 FB15k-sized DistMult steps 3976 -> 3895.
constexpr int REPLAY_SIZES = 2;
constexpr int64_t REPLAY_STEPS[REPLAY_SIZES] = {16, 32};  // (graphs of 64 steps were slower than of 32)
constexpr int64_t REPLAY_LONG = 256;

// What a captured graph depends on.  The id arrays, the per-step sides and the loss array are not part of it: the
// kernels find them through the step block.
struct ReplayKey {
    void *ent, *ent_state, *rel, *rel_state;
    int64_t b, k, chunk;
    float gamma, lr;
    bool operator==(const ReplayKey& o) const { return memcmp(this, &o, sizeof(ReplayKey)) == 0; }
};

struct ReplayCache {
    bool counted = false;  // kge_graph_captures has counted the key
    ReplayKey key = {};
    hipGraphExec_t exec[REPLAY_SIZES] = {};  // exec[i] runs REPLAY_STEPS[i] steps; captured when first needed
};

void replay_drop(ReplayCache* rc) {
    for (int i = 0; i < REPLAY_SIZES; ++i) {
        if (rc->exec[i]) (void)hipGraphExecDestroy(rc->exec[i]);
        rc->exec[i] = nullptr;
    }
    rc->counted = false;
}

// The cache, emptied if it holds graphs of another key; null without host memory.
ReplayCache* replay_cache(kge_ctx* c, float* ent, float* ent_state, float* rel, float* rel_state, int64_t b, int64_t k,
                          int64_t chunk, float gamma, float lr) {
    ReplayKey key;
    memset(&key, 0, sizeof(key));
    key.ent = ent; key.ent_state = ent_state; key.rel = rel; key.rel_state = rel_state;
    key.b = b; key.k = k; key.chunk = chunk; key.gamma = gamma; key.lr = lr;
    if (!c->replay) c->replay = new (std::nothrow) ReplayCache();
    ReplayCache* cache = (ReplayCache*)c->replay;
    if (cache && !(cache->key == key)) {
        replay_drop(cache);
        cache->key = key;
    }
    return cache;
}

// A graph of n steps into *out, which stays null if it cannot be built (that is no error: the steps can be launched
// kernel by kernel).
void capture_steps(kge_ctx* c, float* ent, float* ent_state, float* rel, float* rel_state, const StepIds& ids, int K,
                   int G, float gamma, float lr, hipStream_t st, int n, hipGraphExec_t* out) {
    hipGraph_t graph = nullptr;
    if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) == hipSuccess) {
        int rc = KGE_OK;
        for (int s = 0; s < n && rc == KGE_OK; ++s) rc = enqueue_step(c, ent, ent_state, rel, rel_state, ids, K, G, gamma, lr, st);
        const bool ok = hipStreamEndCapture(st, &graph) == hipSuccess && rc == KGE_OK;
        if (ok && hipGraphInstantiate(out, graph, nullptr, nullptr, 0) != hipSuccess) *out = nullptr;
        if (graph) (void)hipGraphDestroy(graph);
        if (*out) {
            ReplayCache* cache = (ReplayCache*)c->replay;
            if (!cache->counted) c->graph_captures += 1;
            cache->counted = true;
            (void)hipGraphUpload(*out, st);  // so that the first launch does not pay for it; a failure here is not one
        }
    }
    c->err[0] = 0;
    (void)hipGetLastError();
}

// Replays the steps of a call from *done on, at most KGE_SIDES_CAP of them, and moves *done past those that were enqueued;
// true if that was all of them.  (n_steps - *done is a multiple of the graph's `unit` steps, and so is KGE_SIDES_CAP.)
bool replay_segment(kge_ctx* c, const int64_t* h, const int64_t* r, const int64_t* t, int64_t b, const int64_t* neg, int64_t n_neg,
                    const int32_t* neg_sides, int64_t n_steps, float* loss_out, hipGraphExec_t exec, int64_t unit, hipStream_t st,
                    int64_t* done) {
    const int64_t first = *done, n = n_steps - first < KGE_SIDES_CAP ? n_steps - first : KGE_SIDES_CAP;
    StepBlock blk;
    blk.step = 0;
    blk.h = h + first * b; blk.r = r + first * b; blk.t = t + first * b; blk.neg = neg + first * n_neg;
    blk.sides = nullptr;
    blk.side_bits = 0;
    // the sides of a single graph travel as bits of the step block; those of a longer replay live in a fixed part of the
    // workspace
    if (neg_sides && n <= 64) {
        for (int64_t s = 0; s < n; ++s) blk.side_bits |= (uint64_t)(neg_sides[first + s] == KGE_NEG_HEAD) << s;
    } else if (neg_sides) {
        if (hipMemcpyAsync(c->sides_dev, neg_sides + first, sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, st) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        blk.sides = c->sides_dev;
    }
    blk.loss_out = loss_out ? loss_out + first : nullptr;
    kge_launch_set_step_block(c->step_block, blk, st);
    bool ok = hipGetLastError() == hipSuccess;
    for (int64_t q = n / unit; ok && q > 0; --q) {
        ok = hipGraphLaunch(exec, st) == hipSuccess;
        if (ok) *done += unit;
    }
    (void)hipGetLastError();
    return ok;
}

}  // namespace

extern "C" {

int kge_create(const kge_config* cfg, kge_ctx** out) {
    if (!cfg || !out) return fail(nullptr, KGE_ERR_INVALID_ARG, "null argument%s");
    *out = nullptr;
    const int m = cfg->model;
    if (m < KGE_TRANSE_L2 || m > KGE_TRANSR) return fail(nullptr, KGE_ERR_INVALID_ARG, "unknown model%s");
    const bool cplx = m == KGE_COMPLEX || m == KGE_ROTATE;
    if (cfg->ent_dim <= 0 || cfg->ent_dim > 1024 || cfg->ent_dim % (cplx ? 8 : 4) != 0)
        return fail(nullptr, KGE_ERR_INVALID_ARG, "ent_dim must be a multiple of 4 (8 for ComplEx/RotatE), at most 1024%s");
    const int sq = cfg->ent_dim * cfg->ent_dim;
    const int want_rel = m == KGE_ROTATE ? cfg->ent_dim / 2 : (m == KGE_RESCAL ? sq : (m == KGE_TRANSR ? cfg->ent_dim + sq : cfg->ent_dim));
    if (cfg->rel_dim != want_rel)
        return fail(nullptr, KGE_ERR_INVALID_ARG, "rel_dim must be ent_dim (ent_dim/2 for RotatE, ent_dim^2 for RESCAL, ent_dim + ent_dim^2 for TransR)%s");
    if ((m == KGE_RESCAL || m == KGE_TRANSR) && (cfg->adagrad_mode != 0 || cfg->gemm_input != 0))
        return fail(nullptr, KGE_ERR_UNSUPPORTED, "RESCAL and TransR run with element-wise Adagrad state and fp32 operands only%s");
    if (cfg->num_entities <= 0 || cfg->num_relations <= 0 || cfg->num_entities >= (1ll << 32) ||
        cfg->num_relations >= (1ll << 32))
        return fail(nullptr, KGE_ERR_INVALID_ARG, "table row counts must be in [1, 2^32)%s");
    if (cfg->max_batch <= 0 || cfg->max_neg_per_chunk < 0 || cfg->max_chunks <= 0 || cfg->max_chunks > cfg->max_batch)
        return fail(nullptr, KGE_ERR_INVALID_ARG, "bad workspace limits%s");
    if ((int64_t)cfg->max_chunks * cfg->max_neg_per_chunk + 2ll * cfg->max_batch > (1 << 24))
        return fail(nullptr, KGE_ERR_INVALID_ARG, "more than 2^24 entity keys per step%s");
    if (cfg->adagrad_mode != 0 && cfg->adagrad_mode != 1) return fail(nullptr, KGE_ERR_INVALID_ARG, "adagrad_mode must be 0 or 1%s");
    if (cfg->loss != KGE_LOSS_LOGISTIC && cfg->loss != KGE_LOSS_RANKING) return fail(nullptr, KGE_ERR_INVALID_ARG, "loss must be 0 (logistic) or 1 (ranking)%s");
    if (cfg->gemm_input != 0 && cfg->gemm_input != 1) return fail(nullptr, KGE_ERR_INVALID_ARG, "gemm_input must be 0 or 1%s");
    if (cfg->gemm_input == 1 && !is_gemm_model(cfg->model))
        return fail(nullptr, KGE_ERR_UNSUPPORTED, "bf16 operands exist for the matrix-product models only (TransE-L2, DistMult, ComplEx)%s");
    if (cfg->adv_temperature < 0.f || cfg->adagrad_eps < 0.f) return fail(nullptr, KGE_ERR_INVALID_ARG, "negative temperature or eps%s");

    int ndev = 0;
    KGE_HIP(nullptr, hipGetDeviceCount(&ndev));
    if (cfg->device < 0 || cfg->device >= ndev) return fail(nullptr, KGE_ERR_INVALID_ARG, "no such device%s");
    KGE_HIP(nullptr, hipSetDevice(cfg->device));

    kge_ctx* c = new (std::nothrow) kge_ctx();
    if (!c) return fail(nullptr, KGE_ERR_DEVICE, "out of host memory%s");
    memset(c, 0, sizeof(*c));
    c->cfg = *cfg;
    c->eps = cfg->adagrad_eps > 0.f ? cfg->adagrad_eps : 1e-10f;
    c->ld_s = (cfg->max_neg_per_chunk + 3) / 4 * 4;
    if (c->ld_s == 0) c->ld_s = 4;
    c->max_neg_rows = cfg->max_chunks * cfg->max_neg_per_chunk;
    c->max_ent_keys = 2 * cfg->max_batch + c->max_neg_rows;

    const size_t D = cfg->ent_dim, Dr = cfg->rel_dim, B = cfg->max_batch, NR = c->max_neg_rows > 0 ? c->max_neg_rows : 1;
    const size_t EK = c->max_ent_keys;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes); return o; };
    const size_t o_O = take(B * D * 4), o_N = take(NR * D * 4), o_S = take(B * c->ld_s * 4), o_GO = take(B * D * 4);
    const size_t o_Ge = take(EK * D * 4), o_Gr = take(B * (m == KGE_RESCAL ? 2 * D : Dr) * 4);  // RESCAL keeps two factor rows per positive
    const size_t o_fpos = take(B * 4), o_on2 = take(B * 4), o_nn2 = take(NR * 4), o_cpos = take(B * 4);
    const size_t o_rl = take(B * 4), o_idp = take(B * 4);
    const size_t nlp_gemm = (B / 32 + cfg->max_chunks + 1) * ((size_t)cfg->max_neg_per_chunk / 32 + 1);
    const size_t nlp_pair = (B / 8 + cfg->max_chunks + 1) * KGE_PAIR_MAX_PARTS;
    const size_t nlp_transr = m == KGE_TRANSR ? (B + B / 32 + 16) * ((size_t)cfg->max_neg_per_chunk / 64 + 1) : 0;
    size_t nlp = nlp_gemm > nlp_pair ? nlp_gemm : nlp_pair;
    nlp = nlp > nlp_transr ? nlp : nlp_transr;
    const size_t o_nlp = take(nlp * 4);
    const size_t o_ek0 = take(EK * 4), o_ek1 = take(EK * 4), o_ep0 = take(EK * 4), o_ep1 = take(EK * 4);
    const size_t o_rk0 = take(B * 4), o_rk1 = take(B * 4), o_rp0 = take(B * 4), o_rp1 = take(B * 4);
    const size_t o_flags = take(256), o_step = take(256), o_sides = take(sizeof(int32_t) * KGE_SIDES_CAP);
    c->ld_bf = (cfg->ent_dim + 63) / 64 * 64;  // rows start on 128-byte lines: a K block of a row is one line, not two
    const bool bf = cfg->gemm_input == 1;
    const size_t o_Obf = take(bf ? B * c->ld_bf * 2 + 64 : 0), o_Nbf = take(bf ? NR * c->ld_bf * 2 + 64 : 0);
    const bool transr = m == KGE_TRANSR;
    const size_t o_PP = take(transr ? B * D * 4 : 0), o_trg = take(transr ? kge_transr_carve_groups(*cfg, nullptr, &c->tr_groups) : 0);
    auto sort_digits = [](size_t keys) {  // counts of all slices: 8-bit digits, or 10-bit ones of few slices
        const size_t slices = (keys + KGE_SORT_SLICE - 1) / KGE_SORT_SLICE, few = (size_t)KGE_SORT_FEW_SLICES << KGE_SORT_MAX_BITS;
        return slices * 256 > few ? slices * 256 : few;
    };
    const size_t o_sc = take((sort_digits(EK) + sort_digits(B) + ((size_t)2 << KGE_SORT_MAX_BITS)) * 4);
    const bool pair_model = m == KGE_ROTATE || m == KGE_TRANSE_L1;
    const size_t o_rpw = take((EK / 4 + 4) * 4);
    // everything from here on is written before it is read (the fill below leaves it out).  Partial rows: a set of rows of the
    // corrupting entities per 8 positives of a chunk is the most that a launch writes; no more than 256 MB of them, or 8 sets
    // per chunk where those are more (a launch that would need more walks several tiles of positives per workgroup)
    const size_t zeroed = off;
    const size_t K1 = cfg->max_neg_per_chunk > 0 ? cfg->max_neg_per_chunk : 1;
    size_t sets_n = (B / 8 + cfg->max_chunks) * K1 * D;
    const size_t sets_cap = 8 * NR * D > (size_t)64 << 20 ? 8 * NR * D : (size_t)64 << 20;
    sets_n = sets_n < sets_cap ? sets_n : sets_cap;
    const size_t o_ppo = take(pair_model ? KGE_PAIR_MAX_PARTS * B * D * 4 : 0), o_ppn = take(pair_model ? sets_n * 4 : 0);
    const size_t o_P3 = take(transr ? (kge_transr_p_floats(*cfg) + B * K1 * D) * 4 : 0);
    const size_t o_tgo = take(transr ? kge_transr_go_floats(*cfg) * 4 : 0);
    const size_t o_rr = take(m == KGE_RESCAL ? kge_rescal_runs_bytes(*cfg) : 0);
    const size_t o_tbp = take(transr ? kge_transr_back_floats(*cfg) * 4 : 0);
    c->ws_bytes = (int64_t)off;

    hipError_t e = hipMalloc(&c->ws_base, off);
    if (e != hipSuccess) {
        fail(nullptr, KGE_ERR_DEVICE, "hipMalloc(workspace): %s", hipGetErrorString(e));
        delete c;
        return KGE_ERR_DEVICE;
    }
    char* base = (char*)c->ws_base;
    c->O = (float*)(base + o_O); c->Nst = (float*)(base + o_N); c->S = (float*)(base + o_S);
    c->GO = (float*)(base + o_GO); c->Gent = (float*)(base + o_Ge); c->Grel = (float*)(base + o_Gr);
    c->fpos = (float*)(base + o_fpos); c->o_n2 = (float*)(base + o_on2); c->n_n2 = (float*)(base + o_nn2);
    c->cpos = (float*)(base + o_cpos); c->row_loss = (float*)(base + o_rl);
    c->inv_dpos = (float*)(base + o_idp); c->neg_loss_part = (float*)(base + o_nlp);
    c->ekey[0] = (uint32_t*)(base + o_ek0); c->ekey[1] = (uint32_t*)(base + o_ek1);
    c->epos[0] = (uint32_t*)(base + o_ep0); c->epos[1] = (uint32_t*)(base + o_ep1);
    c->rkey[0] = (uint32_t*)(base + o_rk0); c->rkey[1] = (uint32_t*)(base + o_rk1);
    c->rpos[0] = (uint32_t*)(base + o_rp0); c->rpos[1] = (uint32_t*)(base + o_rp1);
    c->Obf = bf ? (uint16_t*)(base + o_Obf) : nullptr;
    c->Nbf = bf ? (uint16_t*)(base + o_Nbf) : nullptr;
    c->PP = transr ? (float*)(base + o_PP) : nullptr;
    c->P3 = transr ? (float*)(base + o_P3) : nullptr;
    if (transr) kge_transr_carve_groups(*cfg, base + o_trg, &c->tr_groups);
    c->tr_go_part = transr ? (float*)(base + o_tgo) : nullptr;
    c->tr_back_part = transr ? (float*)(base + o_tbp) : nullptr;
    c->rescal_runs = m == KGE_RESCAL ? base + o_rr : nullptr;
    c->pair_part_o = pair_model ? (float*)(base + o_ppo) : nullptr;
    c->pair_part_n = pair_model ? (float*)(base + o_ppn) : nullptr;
    c->pair_part_n_floats = pair_model ? (int64_t)sets_n : 0;
    c->sort_counts = (uint32_t*)(base + o_sc);
    c->run_part_w = (float*)(base + o_rpw);
    c->flags = (int*)(base + o_flags);
    c->step_block = (StepBlock*)(base + o_step);
    c->sides_dev = (int32_t*)(base + o_sides);

    // hipMemset on device memory returns before the fill has run (it is queued on the null stream, behind whatever
    // the caller has there), and the streams that callers pass are not ordered against the null stream: without the
    // wait below the fill could land after the first call has written its step block into the workspace.
    bool ok = hipMemset(c->ws_base, 0, zeroed) == hipSuccess;
    ok = ok && hipDeviceSynchronize() == hipSuccess;
    ok = ok && hipStreamCreateWithFlags(&c->side_stream, hipStreamNonBlocking) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        fail(nullptr, KGE_ERR_DEVICE, "stream/event creation failed%s");
        kge_destroy(c);
        return KGE_ERR_DEVICE;
    }
    *out = c;
    return KGE_OK;
}

void kge_destroy(kge_ctx* c) {
    if (!c) return;
    (void)hipSetDevice(c->cfg.device);
    if (c->side_stream) { (void)hipStreamSynchronize(c->side_stream); (void)hipStreamDestroy(c->side_stream); }
    if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
    if (c->ev_join) (void)hipEventDestroy(c->ev_join);
    for (int s = 0; s < KGE_PROF_SLOTS; ++s)
        for (int e = 0; e < 2; ++e)
            if (c->prof_ev[s][e]) (void)hipEventDestroy(c->prof_ev[s][e]);
    if (c->replay) {
        replay_drop((ReplayCache*)c->replay);
        delete (ReplayCache*)c->replay;
    }
    if (c->ws_base) (void)hipFree(c->ws_base);
    delete c;
}

int kge_train_step(kge_ctx* c, float* ent, float* ent_state, float* rel, float* rel_state,
                   const int64_t* h, const int64_t* r, const int64_t* t, int64_t b,
                   const int64_t* neg, int64_t k, int64_t chunk, int32_t neg_side,
                   float gamma, float lr, void* hip_stream, float* loss_out) {
    if (!c) return KGE_ERR_INVALID_ARG;
    c->err[0] = 0;
    if (!ent_state || !rel_state) return fail(c, KGE_ERR_INVALID_ARG, "null optimizer state%s");
    const int rc = check_batch(c, ent, rel, h, r, t, b, neg, k, chunk, neg_side, true);
    if (rc != KGE_OK) return rc;
    KGE_HIP(c, hipSetDevice(c->cfg.device));
    const StepIds ids = direct_ids(h, r, t, (int)b, neg, (int)((b / chunk) * k), neg_side, loss_out);
    return enqueue_step(c, ent, ent_state, rel, rel_state, ids, (int)k, (int)chunk, gamma, lr, (hipStream_t)hip_stream);
}

int kge_train_steps(kge_ctx* c, float* ent, float* ent_state, float* rel, float* rel_state,
                    const int64_t* h, const int64_t* r, const int64_t* t, int64_t b,
                    const int64_t* neg, int64_t k, int64_t chunk, const int32_t* neg_sides, int64_t n_steps,
                    float gamma, float lr, void* hip_stream, float* loss_out) {
    if (!c) return KGE_ERR_INVALID_ARG;
    c->err[0] = 0;
    if (!ent_state || !rel_state) return fail(c, KGE_ERR_INVALID_ARG, "null optimizer state%s");
    if (n_steps < 0) return fail(c, KGE_ERR_INVALID_ARG, "negative step count%s");
    int rc = check_batch(c, ent, rel, h, r, t, b, neg, k, chunk, KGE_NEG_TAIL, true);
    if (rc != KGE_OK) return rc;
    for (int64_t s = 0; neg_sides && s < n_steps; ++s)
        if (neg_sides[s] != KGE_NEG_TAIL && neg_sides[s] != KGE_NEG_HEAD)
            return fail(c, KGE_ERR_INVALID_ARG, "neg_sides entries must be 0 or 1%s");
    if (n_steps == 0) return KGE_OK;
    KGE_HIP(c, hipSetDevice(c->cfg.device));
    hipStream_t st = (hipStream_t)hip_stream;
    const int64_t n_neg = (b / chunk) * k;

    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    (void)hipStreamIsCapturing(st, &cap);
    static const bool replay_enabled = []() {
        const char* e = getenv("KGE_TRAIN_STEPS_REPLAY");  // "0" turns graph replay off (measurement aid)
        return !(e && e[0] == '0');
    }();
    const bool may_replay = replay_enabled && !c->prof_on && cap == hipStreamCaptureStatusNone && st != nullptr &&
                            st != hipStreamLegacy;  // (the legacy default stream cannot be captured)
    // kernel by kernel: the steps first .. last - 1
    auto plain = [&](int64_t first, int64_t last) {
        for (int64_t s = first; s < last; ++s) {
            const StepIds ids = direct_ids(h + s * b, r + s * b, t + s * b, (int)b, neg + s * n_neg, (int)n_neg,
                                           neg_sides ? neg_sides[s] : KGE_NEG_TAIL, loss_out ? loss_out + s : nullptr);
            const int e = enqueue_step(c, ent, ent_state, rel, rel_state, ids, (int)k, (int)chunk, gamma, lr, st);
            if (e != KGE_OK) return e;
        }
        return (int)KGE_OK;
    };
    if (!may_replay || n_steps < REPLAY_STEPS[0]) return plain(0, n_steps);

    const int which = n_steps < 64 ? 0 : 1;
    const int64_t unit = REPLAY_STEPS[which];
    ReplayCache* cache = replay_cache(c, ent, ent_state, rel, rel_state, b, k, chunk, gamma, lr);
    // A call that is shorter than REPLAY_LONG and finds no graph runs without one and builds it when all of its steps are
    // enqueued: 0.2 ms of host work that the GPU does not wait for (first 20-step call of a Freebase-shaped run 947 us with the
    // capture before the last 16 steps, 787 us of plain steps).  A longer one builds it behind its plain start.
    int64_t n_plain = n_steps < REPLAY_LONG ? n_steps - unit : unit + n_steps % unit;
    if (!cache || (!cache->exec[which] && n_steps < REPLAY_LONG)) n_plain = n_steps;
    rc = plain(0, n_plain);
    if (rc != KGE_OK || !cache) return rc;
    if (!cache->exec[which]) {
        StepIds ids = direct_ids(nullptr, nullptr, nullptr, (int)b, nullptr, (int)n_neg, KGE_NEG_TAIL, nullptr);
        ids.blk = c->step_block;
        capture_steps(c, ent, ent_state, rel, rel_state, ids, (int)k, (int)chunk, gamma, lr, st, (int)unit, &cache->exec[which]);
    }
    // Replay what is left; steps whose graph could not be built or started are launched kernel by kernel, so that a call
    // never ends with an error between two of its steps because of a graph.
    int64_t done = n_plain;
    while (done < n_steps && cache->exec[which] && replay_segment(c, h, r, t, b, neg, n_neg, neg_sides, n_steps, loss_out,
                                                                   cache->exec[which], unit, st, &done)) {}
    return plain(done, n_steps);
}

int kge_score(kge_ctx* c, const float* ent, const float* rel,
              const int64_t* h, const int64_t* r, const int64_t* t, int64_t b,
              const int64_t* neg, int64_t k, int64_t chunk, int32_t neg_side, float gamma,
              void* hip_stream, float* pos_out, float* neg_out) {
    if (!c) return KGE_ERR_INVALID_ARG;
    c->err[0] = 0;
    const int rc = check_batch(c, ent, rel, h, r, t, b, neg, k, chunk, neg_side, neg_out != nullptr);
    if (rc != KGE_OK) return rc;
    KGE_HIP(c, hipSetDevice(c->cfg.device));
    const int kk = neg_out ? (int)k : 0;
    const StepIds ids = direct_ids(h, r, t, (int)b, neg, (int)((b / chunk) * kk), neg_side, nullptr);
    forward(c, ent, rel, ids, kk, (int)chunk, gamma, pos_out, neg_out, (int)k, 0, (hipStream_t)hip_stream);
    KGE_HIP(c, hipGetLastError());
    return KGE_OK;
}

int kge_score_noalloc(const kge_config* cfg, const float* ent, const float* rel,
                      const int64_t* h, const int64_t* r, const int64_t* t, int64_t b,
                      const int64_t* neg, int64_t k, int64_t chunk, int32_t neg_side, float gamma,
                      void* hip_stream, float* pos_out, float* neg_out) {
    if (!cfg) return fail(nullptr, KGE_ERR_INVALID_ARG, "null configuration%s");
    const int m = cfg->model;
    if (m != KGE_TRANSE_L2 && m != KGE_TRANSE_L1 && m != KGE_DISTMULT && m != KGE_COMPLEX && m != KGE_ROTATE)
        return fail(nullptr, KGE_ERR_UNSUPPORTED, "kge_score_noalloc serves TransE-L1/L2, DistMult, ComplEx and RotatE%s");
    if (cfg->gemm_input != 0) return fail(nullptr, KGE_ERR_UNSUPPORTED, "kge_score_noalloc takes fp32 operands only%s");
    const bool cplx = m == KGE_COMPLEX || m == KGE_ROTATE;
    if (cfg->ent_dim <= 0 || cfg->ent_dim > 1024 || cfg->ent_dim % (cplx ? 8 : 4) != 0)
        return fail(nullptr, KGE_ERR_INVALID_ARG, "ent_dim must be a multiple of 4 (8 for ComplEx/RotatE), at most 1024%s");
    if (cfg->rel_dim != (m == KGE_ROTATE ? cfg->ent_dim / 2 : cfg->ent_dim))
        return fail(nullptr, KGE_ERR_INVALID_ARG, "rel_dim must be ent_dim (ent_dim/2 for RotatE)%s");
    if (cfg->num_entities <= 0 || cfg->num_relations <= 0 || cfg->num_entities >= (1ll << 32) ||
        cfg->num_relations >= (1ll << 32))
        return fail(nullptr, KGE_ERR_INVALID_ARG, "table row counts must be in [1, 2^32)%s");
    if (!ent || !rel || !h || !r || !t) return fail(nullptr, KGE_ERR_INVALID_ARG, "null table or id pointer%s");
    if (b <= 0 || chunk <= 0 || b % chunk != 0) return fail(nullptr, KGE_ERR_INVALID_ARG, "b must be a positive multiple of chunk%s");
    if (k < 0 || (neg_out && k == 0)) return fail(nullptr, KGE_ERR_INVALID_ARG, "k out of range%s");
    if (neg_out && !neg) return fail(nullptr, KGE_ERR_INVALID_ARG, "neg is null%s");
    if (neg_side != KGE_NEG_TAIL && neg_side != KGE_NEG_HEAD) return fail(nullptr, KGE_ERR_INVALID_ARG, "neg_side must be 0 or 1%s");
    const int64_t kk = neg_out ? k : 0, n_neg = (b / chunk) * kk;
    if (b > (1 << 24) || n_neg > (1 << 24) || kk > (1 << 24)) return fail(nullptr, KGE_ERR_WORKSPACE, "b or (b/chunk)*k beyond 2^24%s");
    // layout of the scratch array for this call: o rows | staged corrupting rows | six small vectors
    const size_t D = (size_t)cfg->ent_dim, B = (size_t)b, NR = (size_t)(n_neg > 0 ? n_neg : 1);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes); return o; };
    const size_t o_O = take(B * D * 4), o_N = take(NR * D * 4), o_fpos = take(B * 4), o_on2 = take(B * 4);
    const size_t o_nn2 = take(NR * 4), o_cpos = take(B * 4), o_idp = take(B * 4), o_rl = take(B * 4);
    if (off > KGE_NOALLOC_SCRATCH_BYTES)
        return fail(nullptr, KGE_ERR_WORKSPACE, "kge_score_noalloc: 4 * ent_dim * (b + (b/chunk)*k) bytes of rows (plus 24 bytes per row) exceed its 8 MiB of scratch memory%s");

    int ndev = 0;
    KGE_HIP(nullptr, hipGetDeviceCount(&ndev));
    if (cfg->device < 0 || cfg->device >= ndev) return fail(nullptr, KGE_ERR_INVALID_ARG, "no such device%s");
    KGE_HIP(nullptr, hipSetDevice(cfg->device));
    void* base_v = nullptr;
    KGE_HIP(nullptr, scratch_address(cfg->device, &base_v));
    char* base = (char*)base_v;

    // a context that lives on this call's stack and owns nothing: its buffers are pieces of the scratch array.
    // Every piece that a kernel of this call reads has been written by an earlier kernel of the same call (the gather
    // launch fills all of them), so nothing has to be cleared between calls.
    kge_ctx c;
    memset(&c, 0, sizeof(c));
    c.cfg = *cfg;
    c.cfg.validate_indices = 0;  // there is no context to report to: ids are clamped into their tables, as always
    c.cfg.adagrad_mode = 0; c.cfg.loss = KGE_LOSS_LOGISTIC; c.cfg.adv_temperature = 0.f;
    c.cfg.max_batch = (int32_t)b; c.cfg.max_neg_per_chunk = (int32_t)kk; c.cfg.max_chunks = (int32_t)(b / chunk);
    c.ld_s = (int)kk;
    c.O = (float*)(base + o_O); c.Nst = (float*)(base + o_N); c.fpos = (float*)(base + o_fpos);
    c.o_n2 = (float*)(base + o_on2); c.n_n2 = (float*)(base + o_nn2); c.cpos = (float*)(base + o_cpos);
    c.inv_dpos = (float*)(base + o_idp); c.row_loss = (float*)(base + o_rl);
    const StepIds ids = direct_ids(h, r, t, (int)b, neg, (int)n_neg, neg_side, nullptr);
    forward(&c, ent, rel, ids, (int)kk, (int)chunk, gamma, pos_out, neg_out, (int)k, 0, (hipStream_t)hip_stream);
    KGE_HIP(nullptr, hipGetLastError());
    return KGE_OK;
}

int kge_rank(kge_ctx* c, const float* ent, const float* rel,
             const int64_t* h, const int64_t* r, const int64_t* t, int64_t b,
             const int64_t* neg, int64_t k, int64_t chunk, int32_t neg_side, float gamma,
             void* hip_stream, int32_t* rank_out) {
    if (!c) return KGE_ERR_INVALID_ARG;
    c->err[0] = 0;
    if (!rank_out) return fail(c, KGE_ERR_INVALID_ARG, "rank_out is null%s");
    const int rc = check_batch(c, ent, rel, h, r, t, b, neg, k, chunk, neg_side, true);
    if (rc != KGE_OK) return rc;
    KGE_HIP(c, hipSetDevice(c->cfg.device));
    const StepIds ids = direct_ids(h, r, t, (int)b, neg, (int)((b / chunk) * k), neg_side, nullptr);
    hipStream_t st = (hipStream_t)hip_stream;
    if (is_gemm_model(c->cfg.model) && kge_gemm_forward_can_rank(c) && !kge_ind_score_fits(c, (int)chunk)) {
        // the gather launch sets every rank to 1, the forward launch adds the candidates that score higher
        c->rank_out = rank_out;
        forward(c, ent, rel, ids, (int)k, (int)chunk, gamma, nullptr, c->S, c->ld_s, 3, st);
        c->rank_out = nullptr;
    } else {
        forward(c, ent, rel, ids, (int)k, (int)chunk, gamma, nullptr, c->S, c->ld_s, 0, st);
        kge_launch_rank(c, (int)b, (int)k, rank_out, st);
    }
    KGE_HIP(c, hipGetLastError());
    return KGE_OK;
}

int kge_rank_metrics(const int32_t* ranks, int64_t n, double* metrics_out, void* hip_stream) {
    if (!ranks || !metrics_out || n <= 0) return fail(nullptr, KGE_ERR_INVALID_ARG, "null pointer or no ranks%s");
    kge_launch_rank_metrics(ranks, n, metrics_out, (hipStream_t)hip_stream);
    if (hipGetLastError() != hipSuccess) return fail(nullptr, KGE_ERR_DEVICE, "launch of the metrics kernel failed%s");
    return KGE_OK;
}

int kge_get_dedup(kge_ctx* c, int32_t which, int64_t* uniq_out, int32_t* count_out, int64_t* n_unique_out,
                  void* hip_stream) {
    if (!c) return KGE_ERR_INVALID_ARG;
    c->err[0] = 0;
    if ((which != 0 && which != 1) || !uniq_out || !count_out || !n_unique_out)
        return fail(c, KGE_ERR_INVALID_ARG, "bad argument to kge_get_dedup%s");
    if (c->last_ent_keys == 0) return fail(c, KGE_ERR_INVALID_ARG, "no training step has run on this context%s");
    KGE_HIP(c, hipSetDevice(c->cfg.device));
    kge_launch_dedup_export(c, which, uniq_out, count_out, n_unique_out, (hipStream_t)hip_stream);
    KGE_HIP(c, hipGetLastError());
    return KGE_OK;
}

int kge_check_indices(kge_ctx* c, void* hip_stream) {
    if (!c) return KGE_ERR_INVALID_ARG;
    c->err[0] = 0;
    KGE_HIP(c, hipSetDevice(c->cfg.device));
    hipStream_t st = (hipStream_t)hip_stream;
    int flag = 0;
    KGE_HIP(c, hipMemcpyAsync(&flag, c->flags, sizeof(int), hipMemcpyDeviceToHost, st));
    KGE_HIP(c, hipStreamSynchronize(st));
    if (flag) {
        KGE_HIP(c, hipMemsetAsync(c->flags, 0, sizeof(int), st));
        KGE_HIP(c, hipStreamSynchronize(st));
        return fail(c, KGE_ERR_INDEX_RANGE, "an id was outside its table%s");
    }
    return KGE_OK;
}

int kge_profile(kge_ctx* c, int32_t enable) {
    if (!c) return KGE_ERR_INVALID_ARG;
    c->err[0] = 0;
    KGE_HIP(c, hipSetDevice(c->cfg.device));
    if (enable && !c->prof_ev[0][0]) {
        for (int s = 0; s < KGE_PROF_SLOTS; ++s)
            for (int e = 0; e < 2; ++e) KGE_HIP(c, hipEventCreate(&c->prof_ev[s][e]));
    }
    c->prof_on = enable != 0;
    for (int s = 0; s < KGE_PROF_SLOTS; ++s) c->prof_ms[s] = 0.0;
    c->prof_steps = 0;
    return KGE_OK;
}

int kge_profile_read(kge_ctx* c, double* ms_out, int64_t* steps_out) {
    if (!c || !ms_out || !steps_out) return KGE_ERR_INVALID_ARG;
    for (int s = 0; s < KGE_PROF_SLOTS; ++s) ms_out[s] = c->prof_ms[s];
    *steps_out = c->prof_steps;
    return KGE_OK;
}

const char* kge_profile_slot_name(int32_t slot) {
    static const char* names[KGE_PROF_SLOTS] = {"gather", "neg_score", "loss", "neg_backward", "chain", "sort", "update", "phi", "rel_update"};
    return slot >= 0 && slot < KGE_PROF_SLOTS ? names[slot] : "";
}

int kge_sample_steps(const kge_sampler* sp, int64_t first_step, int64_t n_steps, int64_t* h, int64_t* r, int64_t* t,
                     int64_t* neg, int32_t* sides, void* stream) {
    if (!sp || !sp->triples || !h || !r || !t) return fail(nullptr, KGE_ERR_INVALID_ARG, "null sampler, triple list or output%s");
    if (sp->n_triples <= 0 || sp->n_triples >= ((int64_t)1 << 32) || sp->num_entities <= 0 ||
        sp->num_entities >= ((int64_t)1 << 32))
        return fail(nullptr, KGE_ERR_INVALID_ARG, "n_triples and num_entities must be in (0, 2^32)%s");
    if (sp->batch <= 0 || sp->n_chunks <= 0 || sp->neg_per_chunk < 0 || sp->n_degree < 0 ||
        sp->n_degree > sp->neg_per_chunk || sp->side_mode < 0 || sp->side_mode > 2)
        return fail(nullptr, KGE_ERR_INVALID_ARG, "batch, n_chunks, neg_per_chunk, n_degree or side_mode out of range%s");
    if (sp->neg_per_chunk > 0 && !neg) return fail(nullptr, KGE_ERR_INVALID_ARG, "neg is null%s");
    if (first_step < 0 || n_steps < 0) return fail(nullptr, KGE_ERR_INVALID_ARG, "negative step range%s");
    if (n_steps == 0) return KGE_OK;
    if (kge_sample_launch(sp, first_step, n_steps, h, r, t, neg, sides, (hipStream_t)stream) != KGE_OK)
        return fail(nullptr, KGE_ERR_DEVICE, "launch of the sampling kernel failed%s");
    return KGE_OK;
}

const char* kge_last_error(const kge_ctx* c) { return c ? c->err : g_create_err; }

int64_t kge_workspace_bytes(const kge_ctx* c) { return c ? c->ws_bytes : 0; }

int64_t kge_graph_captures(const kge_ctx* c) { return c ? c->graph_captures : 0; }

}  // extern "C"
