// RESCAL (Table 1 of the paper): f(h, r, t) = h^T M_r t, with M_r a D x D matrix kept as one relation row of D * D
// floats (row by row).  The split of Sec. 3.3 carries over: with the tail corrupted h^T M n = (M^T h) . n, with the
// head corrupted n^T M t = n . (M t), so with
//     o = M_r^T h   (tail corrupted)        o = M_r t   (head corrupted)
// every score of a positive against a replacement x is o . x, and negative scoring and its backward are the matrix
// products of DistMult.  What is particular to RESCAL is the matrix-vector product on either side of them:
//   k_rescal<false>  o_i from the kept entity and M_r                       (before the gather launch, which then
//                                                                            scores the positive from o_i)
//   k_rescal<true>   the chain rule: with go = dL/do_i (negatives' part from the backward product, plus the
//                    positive pair's dL/df+ * c), the kept entity gets M go (tail corrupted) or M^T go (head), the
//                    replaced entity dL/df+ * o, and the relation the outer product u w^T with (u, w) = (h, go)
//                    (tail) or (go, t) (head).  That would be a gradient row of D * D floats per positive; only its
//                    two factors are stored.
//   k_rescal_update  duplicate reduction and Adagrad for the relation matrices (Sec. 3.1 step 4): for every distinct
//                    relation of the step, dL/dM = sum over its positives of u w^T, formed straight from the factor
//                    rows (2 D floats per positive instead of D * D) and applied to the matrix in place.
// One workgroup per positive.  M is read once, row by row, every row as whole 16-byte loads; the two kinds of
// product are "row dots" (y_r = M[r, :] . v: a wave per row, shuffle reduction) and "column sums"
// (y = sum_r v_r M[r, :]: a thread per 16-byte column slice, rows dealt round-robin to thread groups whose partial
// sums are added in group order).  All sums have a fixed order.
#include "kge_common.h"

namespace {

constexpr int RT = 256;       // threads per workgroup
constexpr int MAX_D = 1024;   // entity rows are at most this long
constexpr int ROWS = 4;       // rows of M per thread and round

struct RescalArgs {
    const float* E;
    const float* R;
    StepIds ids;
    int b, D;
    int64_t n_ent, n_rel;
    float* O;           // [b x D]  phi: written; chain: read
    const float* GO;    // [b x D]  chain: sum_j W_ij n_j
    const float* cpos;  // [b]      chain: dL/df+_i
    float* Gent;        // gradient rows in key order: heads | tails | corrupting rows
    float* GU;          // [b x D]  chain: left factor of the positive's matrix gradient
    float* GW;          // [b x D]  chain: right factor
    const uint32_t* key;  // sorted relation ids of the step and their positions in the mini-batch, where they are there
    const uint32_t* pos;  // already (else null)
};

// Bound by the round trips of the matrix rows: b D^2 floats (164 MB at b 1024, D 200) out of the L2s and the Infinity Cache.  The
// first round is asked for before the vector that it multiplies is there, every further one while the one before is multiplied.
// Where the relation list has been ordered already (the chain rule), an XCD takes a contiguous range of it, so that positives of a
// relation read its matrix from one L2.  50 FB15k-sized steps, us: 6386 -> 6003 (without the order 8 rows per round take 200
// more, 8 rows with it 6266, 16 rows 7312: fewer waves; ordering the list in a launch of its own before phi costs what it gives).
// WIDE: rows of more than 256 floats, whose row dots take several pieces per lane.
template <bool CHAIN, bool WIDE>
__global__ __launch_bounds__(RT) void k_rescal(RescalArgs a) {
    __shared__ __attribute__((aligned(16))) float vec[MAX_D];  // the vector that multiplies M
    __shared__ __attribute__((aligned(16))) float res[MAX_D];  // the product
    __shared__ __attribute__((aligned(16))) float4 part[RT];   // column sums of the thread groups
    const int tid = threadIdx.x, D = a.D, lanes = D / 4;
    const StepView sv = step_view(a.ids);
    int i = blockIdx.x;
    int64_t rid;
    if (a.pos) {  // workgroups go to the XCDs in turn
        const int per_xcd = (a.b + 7) / 8, p = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
        if (p >= a.b) return;
        i = a.pos[p];
        rid = a.key[p];
    } else {
        rid = clamp_id(sv.r[i], a.n_rel);
    }
    const bool head = sv.side == KGE_NEG_HEAD;
    const int64_t hid = clamp_id(sv.h[i], a.n_ent), tl = clamp_id(sv.t[i], a.n_ent);
    const float* pa = a.E + (head ? tl : hid) * (int64_t)D;  // the kept entity
    const float* pc = a.E + (head ? hid : tl) * (int64_t)D;  // the entity that the negatives replace
    const float* M = a.R + rid * (int64_t)D * D;
    const float cp = CHAIN ? a.cpos[i] : 0.f;

    // phi: o = M^T a (tail corrupted: column sums) or M a (head: row dots); the chain rule needs the transposed one
    const bool rowdot = CHAIN ? !head : head;
    const int w = tid >> 6, lane = tid & 63;
    const int groups = RT / lanes, grp = tid / lanes;  // column-slice ownership (lanes <= 256)
    // this thread's piece of a row, its first row and the step to its next (lanes past the row's end read its first piece and
    // add nothing, threads past the last group have no row)
    const int piece = rowdot ? (lane < lanes ? lane : 0) : tid % lanes;
    const int first = rowdot ? w : (grp < groups ? grp : D), step = rowdot ? RT / 64 : groups;
    struct Rows { float4 m[ROWS]; };
    auto load = [&](int r0) {
        Rows x;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) x.m[u] = ld4(M + (int64_t)(r0 + u * step < D ? r0 + u * step : 0) * D + 4 * piece);
        return x;
    };
    Rows x = {};
    if (!WIDE || !rowdot) x = load(first);

    for (int d = tid; d < D; d += RT) vec[d] = CHAIN ? a.GO[(int64_t)i * D + d] + cp * pc[d] : pa[d];
    __syncthreads();

    if (rowdot) {
        float4 vv[WIDE ? 4 : 1];
#pragma unroll
        for (int it = 0; it < (WIDE ? 4 : 1); ++it) {
            const int q = lane + 64 * it;
            vv[it] = q < lanes ? ld4(vec + 4 * q) : f4(0.f);
        }
        if constexpr (!WIDE) {  // one piece per lane
            for (int r0 = first; r0 < D; r0 += ROWS * step) {
                const Rows next = load(r0 + ROWS * step);
#pragma unroll
                for (int u = 0; u < ROWS; ++u) {
                    float s = lane < lanes ? x.m[u].x * vv[0].x + x.m[u].y * vv[0].y + x.m[u].z * vv[0].z + x.m[u].w * vv[0].w : 0.f;
                    s = wave_sum(s);
                    const int r = r0 + u * step;
                    if (lane == 0 && r < D) res[r] = s;
                }
                x = next;
            }
        } else {
            for (int r = w; r < D; r += RT / 64) {
                const float* row = M + (int64_t)r * D;
                float s = 0.f;
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int q = lane + 64 * it;
                    if (q < lanes) {
                        const float4 m = ld4(row + 4 * q);
                        s += m.x * vv[it].x + m.y * vv[it].y + m.z * vv[it].z + m.w * vv[it].w;
                    }
                }
                s = wave_sum(s);
                if (lane == 0) res[r] = s;
            }
        }
    } else {
        float4 y = f4(0.f);
        for (int r0 = first; r0 < D; r0 += ROWS * step) {
            const Rows next = load(r0 + ROWS * step);
#pragma unroll
            for (int u = 0; u < ROWS; ++u) {
                const int r = r0 + u * step;
                const float s = r < D ? vec[r] : 0.f;
                const float4 m = r < D ? x.m[u] : f4(0.f);
                y.x += s * m.x; y.y += s * m.y; y.z += s * m.z; y.w += s * m.w;
            }
            x = next;
        }
        part[tid] = y;
        __syncthreads();
        if (tid < lanes) {
            float4 t = part[tid];
            for (int g = 1; g < groups; ++g) {
                const float4 u = part[g * lanes + tid];
                t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
            }
            st4(res + 4 * tid, t);
        }
    }
    __syncthreads();

    if (!CHAIN) {
        for (int d = tid; d < D; d += RT) a.O[(int64_t)i * D + d] = res[d];
        return;
    }
    // key positions: heads 0 .. b-1, tails b .. 2b-1
    float* ga = a.Gent + (int64_t)(head ? a.b + i : i) * D;
    float* gc = a.Gent + (int64_t)(head ? i : a.b + i) * D;
    for (int d = tid; d < D; d += RT) {
        ga[d] = res[d];
        gc[d] = cp * a.O[(int64_t)i * D + d];
    }
    // dL/dM[r][c] = a_r go_c (tail corrupted, o = M^T a)  or  go_r a_c (head corrupted, o = M a): the factors
    for (int d = tid; d < D; d += RT) {
        a.GU[(int64_t)i * D + d] = head ? vec[d] : pa[d];
        a.GW[(int64_t)i * D + d] = head ? pa[d] : vec[d];
    }
}

struct RescalUpdArgs {
    float* T;             // relation table [n_rel x D*D]
    float* St;            // its Adagrad accumulator
    const uint32_t* key;  // sorted relation ids of the step
    const uint32_t* pos;  // position in the mini-batch of each sorted entry
    int n, D, rows_per_slab;
    int long_y;           // grid rows for the runs of LONG_RUN positives and more
    const float* GU;
    const float* GW;
    float lr, eps;
};

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int LONG_RUN = 16;  // runs of at least this many positives are summed on the matrix cores
constexpr int LT = 32;        // ... in tiles of LT x LT elements of the matrix

// Runs of LONG_RUN positives and more.  dL/dM = U^T W over the run is a matrix product whose inner length is the run:
// a workgroup owns one 32 x 32 tile of the matrix, its four waves take blocks of 16 positives in turn (16 loads in
// flight per lane, straight into fragments: a half-wave's load is 128 consecutive bytes of one factor row), their
// sums meet in LDS in wave order, and Adagrad is applied to the tile.  What this avoids is the serial chain of the
// slabs below, one round of loads per 4 positives (a relation with a quarter of the batch: 64 rounds and more).  From 16
// on because that is the block of positives one wave takes; a shorter run would leave matrix instructions empty and is
// at most four rounds of the slabs.  FB15k-sized, b = 1024, D = 200: 141 -> 132 us per training step; what is left is
// bound by the matrices and their state (192 MB per step).
// Workgroup q looks at sorted position q * LONG_RUN; every long run holds such a position, and the first one in it
// owns the run.
__device__ __forceinline__ void rescal_long_run(const RescalUpdArgs& a, int q, int tile, int tiles, float* red,
                                                uint32_t* lpos, int* first_other) {
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, D = a.D;
    const int m0 = q * LONG_RUN;
    const uint32_t key = a.key[m0];
    if (q > 0 && a.key[m0 - LONG_RUN] == key) return;  // an earlier workgroup's run
    // start: less than LONG_RUN entries back (the entry LONG_RUN back differs or is not there)
    const int back = m0 - 1 - lane;
    const bool other = back < 0 || lane >= LONG_RUN - 1 || a.key[back < 0 ? 0 : back] != key;
    const int start = m0 - __builtin_ctzll(__ballot(other));
    if (start + LONG_RUN > a.n || a.key[start + LONG_RUN - 1] != key) return;  // a short run: the slabs' work
    const int r0 = (tile / tiles) * LT, c0 = (tile % tiles) * LT;
    const int er = r0 + (tid >> 3), ec = c0 + 4 * (tid & 7);  // the elements that this thread updates
    const bool act = er < D && ec < D;
    const int64_t off = (int64_t)key * D * D + (act ? (int64_t)er * D + ec : 0);
    const float4 xin = ld4(a.T + off), sin = ld4(a.St + off);
    const int l = lane & 31, half = lane >> 5;
    const float* gu = a.GU + (r0 + l < D ? r0 + l : D - 1);
    const float* gw = a.GW + (c0 + l < D ? c0 + l : D - 1);
    floatx16 acc = {};
    for (int b0 = start;; b0 += RT) {
        if (tid == 0) *first_other = RT;
        __syncthreads();  // ... and lpos is free again
        const int e = b0 + tid;
        const bool in = e < a.n && a.key[e < a.n ? e : a.n - 1] == key;  // sorted: the run is a prefix of these
        lpos[tid] = in ? a.pos[e] : 0;
        const unsigned long long bal = __ballot(!in);
        if (lane == 0 && bal) atomicMin(first_other, tid + __builtin_ctzll(bal));
        __syncthreads();
        const int m = *first_other;  // positives of the run among these RT
        for (int kb = 16 * w; kb < m; kb += 64) {
            float u[8], v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t row = (int64_t)lpos[kb + 2 * j + half] * D;  // past the end: position 0, dropped below
                u[j] = gu[row];
                v[j] = gw[row];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool live = kb + 2 * j + half < m;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(live ? u[j] : 0.f, live ? v[j] : 0.f, acc, 0, 0, 0);
            }
        }
        __syncthreads();  // everyone has read m
        if (m < RT) break;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) red[w * LT * LT + (8 * (i >> 2) + 4 * half + (i & 3)) * LT + l] = acc[i];
    __syncthreads();
    if (!act) return;
    float4 g = ld4(red + 4 * tid);
#pragma unroll
    for (int k = 1; k < RT / 64; ++k) {
        const float4 t = ld4(red + k * LT * LT + 4 * tid);
        g.x += t.x; g.y += t.y; g.z += t.z; g.w += t.w;
    }
    float4 x = xin, s = sin;
    adagrad4(g, x, s, a.lr, a.eps);
    st4(a.St + off, s);
    st4(a.T + off, x);
}

// Grid: b x (long_y + slabs).  The first long_y rows are (q, tile) of the long runs, which take the longest.  The others
// are (p, slab): if sorted position p is the last of its run of equal relation ids, and the run is shorter than LONG_RUN,
// it owns that relation in this step and updates `rows_per_slab` consecutive rows of its matrix (at most 1024 floats, a
// thread per 16 bytes): the matrix and state slices are asked for first; then the outer products of the run's positives
// are summed in sorted order and Adagrad is applied.  Held to 64 registers: both parts run at full occupancy.
__global__ __launch_bounds__(RT, 8) void k_rescal_update(RescalUpdArgs a) {
    __shared__ __attribute__((aligned(16))) float red[(RT / 64) * LT * LT];
    __shared__ uint32_t lpos[RT];
    __shared__ int first_other;
    const int tid = threadIdx.x, D = a.D;
    if ((int)blockIdx.y < a.long_y) {
        const int tiles = (D + LT - 1) / LT, wg = blockIdx.y * a.n + blockIdx.x, q = wg / (tiles * tiles);
        if (q * LONG_RUN < a.n) rescal_long_run(a, q, wg - q * tiles * tiles, tiles, red, lpos, &first_other);
        return;
    }
    const int p = blockIdx.x, slab = blockIdx.y - a.long_y;
    const uint32_t key = a.key[p];
    if (p + 1 < a.n && a.key[p + 1] == key) return;                    // the run goes on (same decision in every thread)
    if (p + 1 >= LONG_RUN && a.key[p + 1 - LONG_RUN] == key) return;  // a long run
    const int width = a.rows_per_slab * D, lanes = width / 4;
    const bool act = tid < lanes;
    const int e = act ? 4 * tid : 0, lrow = e / D, col = e - lrow * D;
    const int mrow = slab * a.rows_per_slab + lrow;
    const int64_t off = (int64_t)key * D * D + (int64_t)slab * width + e;
    float4 x = f4(0.f), s = f4(0.f);
    if (act) { x = ld4(a.T + off); s = ld4(a.St + off); }
    // lane t of every wave looks at the t-th entry of the run from its end
    const int lane = tid & 63, q = p - lane;
    const bool other = q < 0 || lane >= LONG_RUN || a.key[q < 0 ? 0 : q] != key;
    const int m = __builtin_ctzll(__ballot(other));
    const uint32_t mine = a.pos[q < 0 ? 0 : q];
    float4 g = f4(0.f);
#pragma unroll 4
    for (int j = m - 1; j >= 0; --j) {
        const int64_t row = (int64_t)__builtin_amdgcn_readlane(mine, j) * D;
        const float u = a.GU[row + mrow];
        const float4 w = ld4(a.GW + row + col);
        g.x += u * w.x; g.y += u * w.y; g.z += u * w.z; g.w += u * w.w;
    }
    if (act) {
        adagrad4(g, x, s, a.lr, a.eps);
        st4(a.St + off, s);
        st4(a.T + off, x);
    }
}

RescalArgs make_args(kge_ctx* c, const float* E, const float* R, const StepIds& ids) {
    RescalArgs a = {};
    a.E = E; a.R = R; a.ids = ids; a.b = ids.b; a.D = c->cfg.ent_dim;
    a.n_ent = c->cfg.num_entities; a.n_rel = c->cfg.num_relations;
    a.O = c->O; a.GO = c->GO; a.cpos = c->cpos; a.Gent = c->Gent;
    a.GU = c->Grel; a.GW = c->Grel + (int64_t)ids.b * c->cfg.ent_dim;  // the relation-gradient area holds the factors
    return a;
}

template <bool CHAIN>
void launch_rescal(kge_ctx* c, const RescalArgs& a, hipStream_t st) {
    const dim3 grid(a.pos ? (a.b + 7) / 8 * 8 : a.b);
    if (a.D > 256) KGE_LAUNCH(c, (k_rescal<CHAIN, true>), grid, dim3(RT), 0, st, a);
    else KGE_LAUNCH(c, (k_rescal<CHAIN, false>), grid, dim3(RT), 0, st, a);
}

}  // namespace

void kge_launch_rescal_phi(kge_ctx* c, const float* E, const float* R, const StepIds& ids, hipStream_t st) {
    launch_rescal<false>(c, make_args(c, E, R, ids), st);
}

void kge_launch_rescal_chain(kge_ctx* c, const float* E, const float* R, const StepIds& ids, bool ordered, hipStream_t st) {
    RescalArgs a = make_args(c, E, R, ids);
    if (ordered) { a.key = c->rkey[c->rbuf]; a.pos = c->rpos[c->rbuf]; }
    launch_rescal<true>(c, a, st);
}

void kge_launch_rescal_update(kge_ctx* c, float* R, float* SR, const StepIds& ids, float lr, hipStream_t st) {
    RescalUpdArgs a;
    const int D = c->cfg.ent_dim;
    int rows = 1024 / D;  // matrix rows per workgroup: the largest divisor of D that keeps a slab within 1024 floats
    while (D % rows != 0) --rows;
    a.T = R; a.St = SR; a.key = c->rkey[c->rbuf]; a.pos = c->rpos[c->rbuf];
    a.n = ids.b; a.D = D; a.rows_per_slab = rows;
    a.GU = c->Grel; a.GW = c->Grel + (int64_t)ids.b * D;
    a.lr = lr; a.eps = c->eps;
    const int tiles = (D + LT - 1) / LT;
    a.long_y = ids.b < LONG_RUN ? 0 : (int)(((int64_t)((ids.b + LONG_RUN - 1) / LONG_RUN) * tiles * tiles + ids.b - 1) / ids.b);
    KGE_LAUNCH(c, k_rescal_update, dim3(ids.b, a.long_y + D / rows), dim3(RT), 0, st, a);
}
