// Internal declarations shared by the HIP sources of libkge (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kge.h"
#include <hip/hip_ext.h>

#include "k_pair_plan.h"

// ---------------------------------------------------------------------------------------------------------
// Context.  All device buffers are carved out of one allocation made in kge_create.
//
// Notation (paper Sec. 3.3): b positives per mini-batch, groups ("chunks") of g positives, C = b / g chunks,
// k corrupting entities per chunk, D floats per entity row.  For every positive i the library forms
//     o_i = phi(a_i, r_i)      a_i = the entity that is NOT corrupted (head for tail corruption, else tail)
// so that the score of (i, any replacement x) is psi(o_i, x); this is the split of Sec. 3.3
// (TransE: o = h + r, psi = gamma - |o - x|) carried over to the other models and to head corruption.
// ---------------------------------------------------------------------------------------------------------
// Gradient rows that exist as `parts` partial rows, `stride` floats apart, still to be added up (in order) into out.
struct PartialRows {
    const float* src;
    float* out;
    int parts;       // 0 or 1: nothing to add up
    int64_t stride;
    int64_t n4;      // 16-byte pieces per partial
};

// TransR: the items of a mini-batch, i.e. the (chunk, relation) pairs that occur in it (k_transr.hip).  Item slots of chunk
// c start at c * g; the positives of an item ("members") are numbered consecutively, item after item, chunk after chunk.
struct alignas(16) TransrItem {
    uint32_t rel;
    int off, n;  // members off .. off + n - 1
};
struct alignas(32) TransrBlock {  // up to 32 members of one item
    int slot;
    uint32_t rel;
    int off, n;  // members off .. off + n - 1
    int first;   // number of the item's members before this block
    int all;     // members of the item
};
struct TransrGroups {
    TransrItem* items;     // [b] by slot
    TransrBlock* pblocks;  // per chunk
    int* members;          // [b] by member: position in the mini-batch
    uint32_t* ent;         // [2 b] by member: rows of the kept and the replaced entity
    int* count;            // [b] by member: members of its item
    int* slot_of;          // [b] by position: the item slot if it is the first of its item, else -1
    int* unit_of;          // [b] by position: c * g + e if it is the first of block e of its chunk's blocks, else -1
    int* first;            // [b] by position, long chunks only: first position of the item in the chunk; its rank among those
    int* rank;
    int* n_items;          // [C]
    int* n_pblocks;        // [C]
};

struct StepBlock;

struct kge_ctx {
    kge_config cfg;
    float eps;
    int ld_s;            // row pitch of S / W in floats (max_neg_per_chunk rounded up to 4)
    int max_neg_rows;    // max_chunks * max_neg_per_chunk
    int max_ent_keys;    // 2 * max_batch + max_neg_rows
    int ent_key_bits, rel_key_bits;

    void* ws_base;
    int64_t ws_bytes;

    float* O;        // [max_batch x D]      o_i
    float* Nst;      // [max_neg_rows x D]   gathered corrupting rows, chunk after chunk
    uint16_t* Obf;   // bf16 operands only: o_i and the corrupting rows rounded to bf16, row pitch ld_bf (the products
    uint16_t* Nbf;   // read these; Nst is then not written)
    int ld_bf;       // D rounded up to 64 (rows of whole 128-byte lines)
    float* S;        // [max_batch x ld_s]   negative scores, then backward coefficients W
    float* PP;       // TransR: [max_batch x D] p_i = M_i c_i
    float* P3;       // TransR: [max_batch x max_neg_per_chunk x D] projections of the corrupting rows (where steps keep them); the same of dL/dP
    TransrGroups tr_groups;
    float* tr_go_part;    // TransR: partial sums of dL/do
    float* tr_back_part;  //         partial gradient rows of the corrupting entities
    float* GO;       // [max_batch x D]      dL/do_i
    void* rescal_runs;   // RESCAL: the runs of equal relations of the running step
    float* pair_part_o;  // RotatE / TransE-L1: [KGE_PAIR_MAX_PARTS][max_batch x D] partial dL/do rows
    PartialRows go_partial, neg_partial;  // what the last backward launch left for the chain launch to add up
    float* pair_part_n;  //                     partial rows of the corrupting entities, a set per tile of positives
    int64_t pair_part_n_floats;
    PairBwdPlan pair_plan;  // of the shape that came last
    float* Gent;     // [max_ent_keys x D]   gradient rows in key order: heads | tails | corrupting rows
    float* Grel;     // [max_batch x Dr]     gradient rows of the relations
    float* run_part_w;  // k_update_runs: sums of W that belong to the partial rows of the running step
    float* fpos;     // [max_batch]          positive scores
    float* o_n2;     // [max_batch]          |o_i|^2          (TransE-L2)
    float* n_n2;     // [max_neg_rows]       |n_j|^2          (TransE-L2)
    float* cpos;     // [max_batch]          dL/df+_i
    float* row_loss; // [max_batch]          loss terms of positive i, already divided by b
    float* inv_dpos; // [max_batch]          1 / |o_i - c_i|  (TransE-L2)
    float* neg_loss_part;  // [forward tiles]  negative-side loss sums written by the forward launch
    uint32_t* ekey[2];  // entity sort ping-pong: keys
    uint32_t* epos[2];  //                        positions in the key list
    uint32_t* rkey[2];  // relation sort ping-pong
    uint32_t* rpos[2];
    int* flags;         // [0]: an id was out of range
    int32_t* rank_out;  // kge_rank: where the running call wants the ranks (the gather launch sets them to 1, the
                        // forward launch counts); null otherwise

    int ebuf, rbuf;                 // which ping-pong half holds the sorted result
    uint32_t* sort_counts;          // radix sort: digit counts per slice of both lists, digit bases
    int64_t last_ent_keys, last_rel_keys;  // sizes of the last train step's key lists (0: none yet)
    hipStream_t side_stream;        // runs the key sort beside the forward/backward kernels
    hipEvent_t ev_fork, ev_join;
    StepBlock* step_block;          // device: id arrays and step counter of the running kge_train_steps call
    int32_t* sides_dev;             // device: per-step sides of the running call, KGE_SIDES_CAP entries
    void* replay;                   // cached graphs of kge_train_steps (ReplayCache in kge_api.hip)
    int64_t graph_captures;         // how many times they were built
    bool prof_on;                   // kge_profile: bracket every kernel with events
    hipEvent_t prof_ev[KGE_PROF_SLOTS][2];
    uint32_t prof_launched;         // slots whose events the running step's launches carry
    double prof_ms[KGE_PROF_SLOTS];
    int64_t prof_steps;
    hipEvent_t launch_ev0, launch_ev1;  // set by a profiling scope: the next KGE_LAUNCH takes its own start/stop
                                        // timestamps into them
    char err[512];
};

// Kernel launch.  While profiling, the launch carries a start and a stop event that receive the dispatch's own
// begin / end timestamps (the ones a kernel trace shows), not the time at which a marker between kernels was
// processed.  One timed launch per profiling scope.
#define KGE_LAUNCH(c, kernel, grid, block, lds, st, ...)                                                            \
    do {                                                                                                            \
        if ((c)->launch_ev0) {                                                                                      \
            hipExtLaunchKernelGGL(kernel, grid, block, lds, st, (c)->launch_ev0, (c)->launch_ev1, 0, __VA_ARGS__);  \
            (c)->launch_ev0 = nullptr;                                                                              \
            (c)->launch_ev1 = nullptr;                                                                              \
        } else {                                                                                                    \
            hipLaunchKernelGGL(kernel, grid, block, lds, st, __VA_ARGS__);                                          \
        }                                                                                                           \
    } while (0)

// ---------------------------------------------------------------------------------------------------------
// The ids of one step, as the kernels receive them.
// Direct mode: blk == nullptr and h, r, t, neg point at this step's ids, side and loss_out are this step's.
// Replay mode (one captured HIP graph serves every step of every kge_train_steps call of the same shape): blk points
// at a block in the workspace that a one-thread kernel fills at the start of every call with the call's id arrays
// (ids of its step 0; consecutive steps lie b (n_neg) entries apart), its per-step sides and its loss array (one float per
// step, may be null), and whose step counter the last
// kernel of every step advances.  The graphs hold only the block's address, so new id arrays need no new capture.
// ---------------------------------------------------------------------------------------------------------
struct StepBlock {
    int64_t step;
    const int64_t* h;
    const int64_t* r;
    const int64_t* t;
    const int64_t* neg;
    const int32_t* sides;   // null: the sides are side_bits (of up to 64 steps; 0: tail corruption throughout)
    uint64_t side_bits;
    float* loss_out;
};

struct StepIds {
    const int64_t* h;
    const int64_t* r;
    const int64_t* t;
    const int64_t* neg;
    int b, n_neg, side;
    StepBlock* blk;
    float* loss_out;
};

// A key list of the duplicate reduction: the concatenation of up to three id arrays (entities: heads | tails |
// corrupting ids; relations: r), to be brought into (id, position) order.
struct KeyList {
    const int64_t* src[3];   // direct mode
    int n_src[3];
    const StepBlock* blk;    // replay mode: the arrays come from the block (which == 0: h | t | neg, 1: r)
    int which;
    int n;                   // total number of keys
    int passes, digit_bits;  // radix passes needed for ids < n_ids, bits per pass
    int64_t n_ids;           // ids are clamped into [0, n_ids)
    uint32_t* key[2];        // sorted ids (ping-pong halves; the rank path writes half 0)
    uint32_t* pos[2];        // position in the key list of each sorted entry
};
// Workgroups of 256 threads for sum_partial_rows and the threads that share a piece: 16 bytes of 8 partial rows or more per
// thread; a thread per piece where that already makes 2048 workgroups, which then take up to four rounds each.
inline int partial_rows_blocks(const PartialRows& r, int& share) {
    share = 1;
    if (r.parts <= 1) return 0;
    while (share < 16 && r.parts > 8 * share && r.n4 * share < 2048 * 256) share *= 2;
    const int64_t blocks = (r.n4 * share + 255) / 256;
    return (int)(blocks <= 2048 ? blocks : (blocks + 3) / 4 > 2048 ? (blocks + 3) / 4 : 2048);
}
void kge_make_key_lists(kge_ctx* c, const StepIds& ids, KeyList* ent, KeyList* rel);

// Grids of more workgroups than one dimension takes (less than 2^32 threads): rows of 2^20, in the order of flat_block().
// What comes behind the last workgroup in the last row has to end at once.
inline dim3 flat_grid(int64_t blocks) {
    const int64_t row = (int64_t)1 << 20;
    return blocks <= row ? dim3((unsigned)blocks) : dim3((unsigned)row, (unsigned)((blocks + row - 1) / row));
}

// ---------------------------------------------------------------------------------------------------------
// Host-side launchers (each in the source file named after its kernel group)
// ---------------------------------------------------------------------------------------------------------
// a1/a2: gather rows, o_i, positive scores, norms
// with_keys: the same launch also brings the key lists into (id, position) order (lists of up to
// KGE_RANK_MAX_KEYS keys; longer lists go through kge_launch_sort)
// (TransR: and the items of the chunks of g positives)
void kge_launch_gather(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int g, float gamma, float* pos_out,
                       bool with_keys, hipStream_t st);
// ... and a3 in the same launch, where the output has few tiles
bool kge_front_fits(const kge_ctx* c, int b, int k, int g, bool with_keys);
void kge_launch_front(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, int g, float gamma, float* pos_out,
                      bool train, bool with_keys, float* out, int ld_out, int out_mode, hipStream_t st);
void kge_launch_key_order(kge_ctx* c, const StepIds& ids, hipStream_t st);  // the key lists alone
// chunks of one positive: everything between the ids and the gradient rows of the positives in one launch, and the
// update of the entity rows that forms the corrupting rows' gradients itself
bool kge_ind_step_fits(const kge_ctx* c, int g);
bool kge_ind_score_fits(const kge_ctx* c, int g);
void kge_ind_step(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, float gamma, hipStream_t st);
void kge_ind_score(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, float gamma, float* out,
                   int ld_out, float* pos_out, hipStream_t st);
void kge_launch_update_runs(kge_ctx* c, float* E, float* SE, const StepIds& ids, int k, float lr, hipStream_t st);
constexpr int KGE_SIDES_CAP = 65536;  // steps whose sides fit the workspace: longer kge_train_steps calls run in segments
constexpr int KGE_SORT_SLICE = 2048;     // keys per workgroup of the radix sort of long key lists
constexpr int KGE_SORT_MAX_BITS = 10;    // bits per digit where a list has at most KGE_SORT_FEW_SLICES slices (else 8)
constexpr int KGE_SORT_FEW_SLICES = 32;
constexpr int KGE_RANK_MAX_KEYS = 14336;  // 14 * 1024: positions fit 14 bits, the list and its tables fit 64 KB of LDS
// a3: negative scores of every chunk into out[b x ld_out]: matrix-product models / elementwise-reduce models
void kge_gemm_neg_score(kge_ctx* c, int b, int k, int g, float gamma, float* out, int ld_out, int dist_mode,
                        hipStream_t st);
void kge_pair_neg_score(kge_ctx* c, int b, int k, int g, float gamma, float* out, int ld_out, hipStream_t st);
// a4: loss terms and backward coefficients (in place over S)
void kge_launch_loss(kge_ctx* c, int b, int k, float gamma, hipStream_t st);
// a5: dL/do and the gradient rows of the corrupting entities
void kge_gemm_neg_backward(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, int g, float gamma,
                           hipStream_t st);
bool kge_gemm_forward_can_rank(const kge_ctx* c);  // evaluation without storing the scores (fp32 products)
bool kge_gemm_backward_forms_w(const kge_ctx* c);     // the forward launch stores W and the loss sums (no k_loss)
bool kge_gemm_backward_does_chain(const kge_ctx* c);  // the backward launch writes the positives' gradient rows
int kge_gemm_loss_parts(const kge_ctx* c, int b, int k, int g);  // loss sums the forward launch leaves in neg_loss_part
// (also a4: returns how many loss sums the launch leaves in neg_loss_part)
int kge_pair_neg_backward(kge_ctx* c, int b, int k, int g, float gamma, hipStream_t st);
// a5: positive-pair term and chain rule through phi -> gradient rows of heads, tails and relations
void kge_launch_chain(kge_ctx* c, const float* E, const float* R, const StepIds& ids, hipStream_t st);
// RESCAL: o_i from the kept entity and the relation's matrix (before the gather launch); chain rule through it
void kge_launch_rescal_phi(kge_ctx* c, const float* E, const float* R, const StepIds& ids, hipStream_t st);
// ordered: the key lists have been ordered on this stream.  By runs (rows of 148 to 256 floats): they have to be, and
// kge_launch_rescal_update does the chain rule of relations of few positives
bool kge_rescal_chain_by_runs(const kge_ctx* c);
size_t kge_rescal_runs_bytes(const kge_config& cfg);
void kge_launch_rescal_chain(kge_ctx* c, const float* E, float* R, const StepIds& ids, bool ordered, hipStream_t st);
// RESCAL, a7 for the relation matrices: gradient of a distinct relation formed from the factor rows, then Adagrad
void kge_launch_rescal_update(kge_ctx* c, const float* E, float* R, float* SR, const StepIds& ids, float lr, hipStream_t st);
// TransR (k_transr.hip)
constexpr int KGE_TRANSR_BACK_WGS = 768, KGE_TRANSR_UNIT_WGS = 256;  // three per CU; one
size_t kge_transr_carve_groups(const kge_config& cfg, char* base, TransrGroups* q);
size_t kge_transr_back_floats(const kge_config& cfg);
size_t kge_transr_go_floats(const kge_config& cfg);
size_t kge_transr_p_floats(const kge_config& cfg);
void kge_transr_phi(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int g, float gamma, float* pos_out,
                    bool train, bool form_w, hipStream_t st);
// train: keep the projections, rows in the order of the members; form_w: store W = dL/df- instead of the scores, returns the number of loss sums left
int kge_transr_project(kge_ctx* c, const float* R, const StepIds& ids, int k, int g, float gamma, float* out, int ld_out,
                       bool train, bool form_w, hipStream_t st);
void kge_transr_dp(kge_ctx* c, const StepIds& ids, int k, int g, bool form_w, hipStream_t st);  // (form_w as in kge_transr_project)
void kge_transr_back(kge_ctx* c, const float* R, const StepIds& ids, int k, int g, bool form_w, hipStream_t st);
void kge_transr_mgrad(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, int g, bool form_w, hipStream_t st);
void kge_transr_update(kge_ctx* c, float* R, float* SR, const StepIds& ids, float lr, bool form_w, hipStream_t st);
// a6: sort (id, position) of the entity and relation key lists
void kge_launch_sort(kge_ctx* c, const StepIds& ids, hipStream_t st);
// a7: per distinct row, sum its gradient rows and apply Adagrad; also reduces the loss terms
// (with_entities: false leaves the entity rows to kge_launch_update_runs)
void kge_launch_update(kge_ctx* c, float* E, float* SE, float* R, float* SR, const StepIds& ids, float lr,
                       int n_loss_parts, bool with_entities, hipStream_t st);
// fills the step block that replayed steps read
void kge_launch_set_step_block(StepBlock* blk, const StepBlock& value, hipStream_t st);
// evaluation: ranks of the positives among their negatives (from fpos and the scores in S), and the metrics
void kge_launch_rank(kge_ctx* c, int b, int k, int32_t* rank_out, hipStream_t st);
void kge_launch_rank_metrics(const int32_t* ranks, int64_t n, double* out, hipStream_t st);
// step 1: ids of a range of steps from the counter-based generator
int kge_sample_launch(const kge_sampler* s, int64_t first_step, int64_t n_steps, int64_t* h, int64_t* r, int64_t* t,
                      int64_t* neg, int32_t* sides, hipStream_t st);
// test hook: distinct ids and multiplicities from the sorted keys
void kge_launch_dedup_export(kge_ctx* c, int which, int64_t* uniq, int32_t* count, int64_t* n_unique,
                             hipStream_t st);

// ---------------------------------------------------------------------------------------------------------
// Device helpers
// ---------------------------------------------------------------------------------------------------------
#ifdef __HIPCC__
struct StepView {
    const int64_t* h;
    const int64_t* r;
    const int64_t* t;
    const int64_t* neg;
    int side;
    int64_t step;
};
__device__ __forceinline__ StepView step_view(const StepIds& s) {
    StepView v;
    if (s.blk) {
        const StepBlock* k = s.blk;  // uniform address: these are scalar loads of one cache line
        v.step = k->step;
        v.h = k->h + v.step * s.b;
        v.r = k->r + v.step * s.b;
        v.t = k->t + v.step * s.b;
        v.neg = k->neg + v.step * s.n_neg;
        const int32_t* sides = k->sides;
        v.side = sides ? sides[v.step] : (int)(k->side_bits >> (v.step & 63) & 1);
    } else {
        v.step = 0;
        v.h = s.h; v.r = s.r; v.t = s.t; v.neg = s.neg;
        v.side = s.side;
    }
    return v;
}
// The (up to three) id arrays of a key list for the running step.
struct KeySources { const int64_t* p[3]; };
__device__ __forceinline__ KeySources key_sources(const KeyList& l) {
    KeySources s;
    if (l.blk) {
        const StepBlock* k = l.blk;
        const int64_t step = k->step;
        if (l.which == 0) {
            s.p[0] = k->h + step * l.n_src[0];
            s.p[1] = k->t + step * l.n_src[1];
            s.p[2] = k->neg + step * l.n_src[2];
        } else {
            s.p[0] = s.p[1] = s.p[2] = k->r + step * l.n_src[0];
        }
    } else {
        s.p[0] = l.src[0]; s.p[1] = l.src[1]; s.p[2] = l.src[2];
    }
    return s;
}
// Address of entry idx of a key list (branch-free, so that a thread can have many of these loads in flight).
__device__ __forceinline__ const int64_t* key_address(const KeyList& l, const KeySources& s, int idx) {
    const int a = l.n_src[0], ab = a + l.n_src[1];
    const int64_t* p0 = s.p[0] + idx;
    const int64_t* p1 = s.p[1] + (idx - a);
    const int64_t* p2 = s.p[2] + (idx - ab);
    return idx < a ? p0 : (idx < ab ? p1 : p2);
}
__device__ __forceinline__ int64_t clamp_id(int64_t id, int64_t n) { return id < 0 ? 0 : (id >= n ? n - 1 : id); }
__device__ __forceinline__ uint32_t clamp_key(const KeyList& l, int64_t id) {
    id = id < 0 ? 0 : (id >= l.n_ids ? l.n_ids - 1 : id);
    return (uint32_t)id;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void st4(float* p, float4 v) { *reinterpret_cast<float4*>(p) = v; }
__device__ __forceinline__ float4 f4(float x) { return make_float4(x, x, x, x); }
__device__ __forceinline__ int flat_block() { return blockIdx.y * gridDim.x + blockIdx.x; }

// sum of `parts` 16-byte pieces `stride` floats apart, in order; eight of them are asked for before the first is added (a
// part that does not exist is read from part 0 and left out of the sum)
__device__ __forceinline__ float4 sum_parts(const float* p, int parts, int64_t stride) {
    if (parts <= 1) return ld4(p);  // (the same for every thread)
    float4 s = f4(0.f);
    for (int q0 = 0; q0 < parts; q0 += 8) {
        float4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = ld4(p + (q0 + q < parts ? q0 + q : 0) * stride);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q0 + q < parts) { s.x += v[q].x; s.y += v[q].y; s.z += v[q].z; s.w += v[q].w; }
        }
    }
    return s;
}

// Partial gradient rows -> their sums, by workgroup `block` of `blocks`: `share` threads per 16 bytes, each a contiguous
// range of the partial rows; their sums meet in LDS in order.
template <int THREADS>
__device__ __forceinline__ void sum_partial_rows(const PartialRows& r, int share, int block, int blocks) {
    __shared__ __attribute__((aligned(16))) float4 sums[THREADS];
    const int cols = THREADS / share, per = (r.parts + share - 1) / share;
    const int grp = threadIdx.x / cols, ln = threadIdx.x % cols;
    const int q0 = grp * per, n = min(per, r.parts - q0);
    for (int64_t e0 = (int64_t)block * cols; e0 < r.n4; e0 += (int64_t)blocks * cols) {
        const int64_t e = e0 + ln;
        float4 s = f4(0.f);
        if (e < r.n4 && n > 0) s = sum_parts(r.src + q0 * r.stride + 4 * e, n, r.stride);
        if (share == 1) {
            if (e < r.n4) st4(r.out + 4 * e, s);
            continue;
        }
        __syncthreads();
        sums[threadIdx.x] = s;
        __syncthreads();
        if (grp == 0 && e < r.n4) {
            for (int g2 = 1; g2 < share; ++g2) {
                const float4 v = sums[g2 * cols + ln];
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            }
            st4(r.out + 4 * e, s);
        }
    }
}

// Adagrad: S += g^2 ; x -= lr * g / (sqrt(S) + eps), with the hardware square root and reciprocal (1 ulp each): the
// update is a step of size <= lr, so their 1e-7 relative error is far below the accuracy of g itself.
__device__ __forceinline__ float adagrad1(float g, float& s, float lr, float eps) {
    s = fmaf(g, g, s);
    return lr * g * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(s) + eps);
}
__device__ __forceinline__ void adagrad4(float4 g, float4& x, float4& s, float lr, float eps) {
    x.x -= adagrad1(g.x, s.x, lr, eps);
    x.y -= adagrad1(g.y, s.y, lr, eps);
    x.z -= adagrad1(g.z, s.z, lr, eps);
    x.w -= adagrad1(g.w, s.w, lr, eps);
}

// fp32 -> bf16 -> fp32, round to nearest even (the hardware conversion of gfx950)
__device__ __forceinline__ float round_bf16(float x) { return (float)(__bf16)x; }
#endif
