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
//   k_rescal_chain_runs, k_rescal_runs  the chain rule and the update for rows of 148 to 256 floats, by runs of positives of a
//                    relation: the first serves relations of 16 positives and more, the second reads the matrices of the
//                    others once for both.
// k_rescal: one workgroup per positive.  M is read once, row by row, every row as whole 16-byte loads; the two kinds of
// product are "row dots" (y_r = M[r, :] . v: a wave per row, shuffle reduction) and "column sums"
// (y = sum_r v_r M[r, :]: a thread per 16-byte column slice, rows dealt round-robin to thread groups whose partial
// sums are added in group order).  All sums have a fixed order.
#include "kge_common.h"

namespace {

constexpr int RT = 256;       // threads per workgroup
constexpr int MAX_D = 1024;   // entity rows are at most this long
constexpr int ROWS = 4;       // rows of M per thread and round
constexpr int LONG_RUN = 16;  // runs of at least this many positives of a relation are products on tiles of their own (below)
constexpr int RUNS_MIN_D = 148, RUNS_D = 256;  // rows of k_rescal_runs (see there)

struct RescalRun { uint32_t key; int first, n; };  // sorted positions first .. first + n - 1 (n: of short runs only)
struct RescalRuns { int count[2], pad[2]; };       // short and long ones; behind it two lists of b runs

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
    RescalArgs chain;  // by runs: of the chain rule
    RescalRuns* runs;
};

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int LT = 32;        // ... in tiles of LT x LT elements of the matrix

// Runs of LONG_RUN positives and more.  dL/dM = U^T W over the run is a matrix product whose inner length is the run:
// a workgroup owns one 32 x 32 tile of the matrix, its waves (four, in k_rescal_runs eight) take blocks of 16 positives in turn (16 loads in
// flight per lane, straight into fragments: a half-wave's load is 128 consecutive bytes of one factor row), their
// sums meet in LDS in wave order, and Adagrad is applied to the tile.  What this avoids is the serial chain of the
// slabs below, one round of loads per 4 positives (a relation with a quarter of the batch: 64 rounds and more).  From 16
// on because that is the block of positives one wave takes; a shorter run would leave matrix instructions empty and is
// at most four rounds of the slabs.  FB15k-sized, b = 1024, D = 200: 141 -> 132 us per training step; what is left is
// bound by the matrices and their state (192 MB per step).
template <int THREADS>
__device__ __forceinline__ void rescal_long_run(const RescalUpdArgs& a, uint32_t key, int start, int tile, int tiles, float* red,
                                                uint32_t* lpos, int* first_other) {
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, D = a.D;
    const int r0 = (tile / tiles) * LT, c0 = (tile % tiles) * LT;
    const int er = r0 + (tid >> 3), ec = c0 + 4 * (tid & 7);  // the elements that this thread updates
    const bool act = tid < LT * LT / 4 && er < D && ec < D;
    const int64_t off = (int64_t)key * D * D + (act ? (int64_t)er * D + ec : 0);
    const float4 xin = ld4(a.T + off), sin = ld4(a.St + off);
    const int l = lane & 31, half = lane >> 5;
    const float* gu = a.GU + (r0 + l < D ? r0 + l : D - 1);
    const float* gw = a.GW + (c0 + l < D ? c0 + l : D - 1);
    floatx16 acc = {};
    for (int b0 = start;; b0 += THREADS) {
        if (tid == 0) *first_other = THREADS;
        __syncthreads();  // ... and lpos is free again
        const int e = b0 + tid;
        const bool in = e < a.n && a.key[e < a.n ? e : a.n - 1] == key;  // sorted: the run is a prefix of these
        lpos[tid] = in ? a.pos[e] : 0;
        const unsigned long long bal = __ballot(!in);
        if (lane == 0 && bal) atomicMin(first_other, tid + __builtin_ctzll(bal));
        __syncthreads();
        const int m = *first_other;  // positives of the run among these THREADS
        for (int kb = 16 * w; kb < m; kb += THREADS / 4) {
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
        if (m < THREADS) break;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) red[w * LT * LT + (8 * (i >> 2) + 4 * half + (i & 3)) * LT + l] = acc[i];
    __syncthreads();
    if (!act) return;
    float4 g = ld4(red + 4 * tid);
#pragma unroll
    for (int k = 1; k < THREADS / 64; ++k) {
        const float4 t = ld4(red + k * LT * LT + 4 * tid);
        g.x += t.x; g.y += t.y; g.z += t.z; g.w += t.w;
    }
    float4 x = xin, s = sin;
    adagrad4(g, x, s, a.lr, a.eps);
    st4(a.St + off, s);
    st4(a.T + off, x);
}

// Where a long run that workgroup q owns starts, or -1.  q looks at sorted position q * LONG_RUN; every long run holds such a
// position, and the first one in it owns the run.
__device__ __forceinline__ int find_long_run(const RescalUpdArgs& a, int q) {
    const int lane = threadIdx.x & 63, m0 = q * LONG_RUN;
    const uint32_t key = a.key[m0];
    if (q > 0 && a.key[m0 - LONG_RUN] == key) return -1;  // an earlier workgroup's run
    // start: less than LONG_RUN entries back (the entry LONG_RUN back differs or is not there)
    const int back = m0 - 1 - lane;
    const bool other = back < 0 || lane >= LONG_RUN - 1 || a.key[back < 0 ? 0 : back] != key;
    const int start = m0 - __builtin_ctzll(__ballot(other));
    return start + LONG_RUN > a.n || a.key[start + LONG_RUN - 1] != key ? -1 : start;  // a short run: the slabs' work
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
        const int start = q * LONG_RUN < a.n ? find_long_run(a, q) : -1;
        if (start >= 0) rescal_long_run<RT>(a, a.key[start], start, wg - q * tiles * tiles, tiles, red, lpos, &first_other);
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

constexpr int PT = 512;           // threads per workgroup
constexpr int KEPT = 32;          // k_rescal_runs: elements of the kept entity per workgroup
constexpr int GP = RUNS_D + 4;    // row pitch of dL/do in LDS
constexpr int RUN_TILES = RUNS_D / 16 / (PT / 64);  // tiles of 16 contracted indices per wave
constexpr int RUNS_LDS = LONG_RUN * GP + LONG_RUN * KEPT + PT / 64 * LONG_RUN * KEPT;  // floats
static_assert(RUNS_LDS >= PT / 64 * LT * LT + PT, "long runs share the memory");

// Up to LONG_RUN positives of one relation, m from sorted position p on, and KEPT elements n of the kept entity: the part of the
// matrix that meets them is KEPT of its rows (tail corrupted) or columns (head), all of them as long as the contracted index x,
//     y_j[n] = sum_x M[n, x] go_j[x]         (the kept entity's gradient)
//     G[n, x] = sum_j a_j[n] go_j[x]         (the matrix's)
// so that a workgroup that holds this part in registers does both, and Adagrad, from one read of it (UPDATE: the m positives are
// all that the relation has; without it y and the factor rows).  Bound by memory: matrices and state, 235 MB per step at b 1024,
// D 200 on the FB15k-sized graph, in 58 us (4.1 TB/s; a large copy reaches 5.2 to 6.0); with the longer runs' chain rule (7) in place of
// the chain rule positive by positive (17) and an update of the matrices alone (55).  512 threads and 78 registers (three workgroups per CU): with 256 threads and
// four tiles per wave 62 us, with 64 columns per workgroup 66, with 64 registers (spills) 72, as workgroups that stay 75.
// A wave takes tiles of 16 x; lane (q, l) holds n = 2 l + c, x = 4 q + i of each, which is the layout of a B operand of
// v_mfma_f32_16x16x4_f32 for the first product (k = q, instruction i) and that of the result of the second (row 4 q + i, column l).
// ids_of(j, m, i, hid, tl, cp): position in the mini-batch, entities and dL/df+ of the j-th of m positives for lanes 0 .. 31, of the next one for
// the others (where there is none: something valid).
template <bool HEAD, bool UPDATE, bool STREAM, class Ids>
__device__ __forceinline__ void rescal_run_part(const RescalUpdArgs& a, Ids ids_of, uint32_t key, int m, int slab, float* lds) {
    const RescalArgs& r = a.chain;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l = lane & 15, q = lane >> 4, D = a.D;
    const int n0 = slab * KEPT, n = n0 + 2 * l, per = ((D + 15) / 16 + PT / 64 - 1) / (PT / 64), x0 = 16 * w * per;
    float* go = lds;                         // [LONG_RUN][GP]
    float* ke = go + LONG_RUN * GP;          // [LONG_RUN][KEPT]
    float* part = ke + LONG_RUN * KEPT;      // [waves][LONG_RUN][KEPT]

    // offsets in bytes, 32 bits: a matrix has up to 256 KB
    struct Tile { float v[2][4]; };
    auto at = [](const float* base, uint32_t off) { return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + off); };
    auto to = [](float* base, uint32_t off) { return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + off); };
    auto load = [&](const float* base, int t) {
        const uint32_t x = x0 + 16 * t + 4 * q, xs = x < (uint32_t)D ? x : 0, ns = n < D ? n : 0;
        Tile f;
        if (HEAD) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 v = *reinterpret_cast<const float2*>(at(base, 4 * ((xs + e) * D + ns)));
                f.v[0][e] = v.x; f.v[1][e] = v.y;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float4 v = ld4(at(base, 4 * ((ns + c) * D + xs)));
                f.v[c][0] = v.x; f.v[c][1] = v.y; f.v[c][2] = v.z; f.v[c][3] = v.w;
            }
        }
        return f;
    };
    float* const T = a.T + (int64_t)key * D * D;
    float* const St = a.St + (int64_t)key * D * D;
    Tile M[RUN_TILES], S[RUN_TILES];
#pragma unroll
    for (int t = 0; t < RUN_TILES; ++t)
        if (t < per) M[t] = load(T, t);
#pragma unroll
    for (int t = 0; UPDATE && t < RUN_TILES; ++t)
        if (t < per) S[t] = load(St, t);

    // a wave stages two positives, 32 lanes each
    const int j = 2 * w + (lane >> 5), s32 = lane & 31;
    const bool live = j < m;
    int64_t i = 0, hid = 0, tl = 0;
    float cp = 0.f;
    if (2 * w < m) {
        ids_of(2 * w, m, i, hid, tl, cp);
        const float* pa = r.E + (HEAD ? tl : hid) * (int64_t)D;
        const float* pc = r.E + (HEAD ? hid : tl) * (int64_t)D;
        float4 g4[2], c4[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int d = 4 * (s32 + 32 * u), ds = d < D ? d : 0;
            g4[u] = ld4(r.GO + i * D + ds);
            c4[u] = ld4(pc + ds);
        }
        const int kn = n0 + 4 * (s32 & 7);
        const bool kin = s32 < 8 && kn < D;
        const float4 ka = ld4(pa + (kin ? kn : 0)), ko = ld4(r.O + i * D + (kin ? kn : 0));
#pragma unroll
        for (int u = 0; u < 2; ++u) {  // (past the row's end and past the run: zeros)
            const int d = 4 * (s32 + 32 * u);
            float4 v = g4[u];
            v.x += cp * c4[u].x; v.y += cp * c4[u].y; v.z += cp * c4[u].z; v.w += cp * c4[u].w;
            st4(go + j * GP + d, live && d < D ? v : f4(0.f));
        }
        if (s32 < 8) st4(ke + j * KEPT + 4 * s32, live && kin ? ka : f4(0.f));
        if (live && kin) {
            st4(r.Gent + (HEAD ? i : r.b + i) * D + kn, make_float4(cp * ko.x, cp * ko.y, cp * ko.z, cp * ko.w));
            if (!UPDATE) st4((HEAD ? r.GW : r.GU) + i * D + kn, ka);
        }
    } else {
#pragma unroll
        for (int u = 0; u < 2; ++u) st4(go + j * GP + 4 * (s32 + 32 * u), f4(0.f));
        if (s32 < 8) st4(ke + j * KEPT + 4 * s32, f4(0.f));
    }
    __syncthreads();

    floatx4 y[2] = {};  // (sums of 4 products at a time, added up in a tree: as exact as sums over the lanes of a wave)
#pragma unroll
    for (int t = 0; t < RUN_TILES; ++t) {
        if (t >= per) break;
        const int x = x0 + 16 * t + 4 * q;
        const float4 f = ld4(go + l * GP + (x < D ? x : 0));
        const float fa[4] = {f.x, f.y, f.z, f.w};
        floatx4 s[2][2];
#pragma unroll
        for (int e = 0; e < 4; e += 2)
#pragma unroll
            for (int c = 0; c < 2; ++c) {  // (both factors: an infinite element of the matrix that is read in a missing one's place)
                const floatx4 s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x < D ? fa[e] : 0.f, x < D ? M[t].v[c][e] : 0.f, floatx4{}, 0, 0, 0);
                const floatx4 s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x < D ? fa[e + 1] : 0.f, x < D ? M[t].v[c][e + 1] : 0.f, floatx4{}, 0, 0, 0);
                s[e / 2][c] = s0 + s1;
            }
#pragma unroll
        for (int c = 0; c < 2; ++c) y[c] += s[0][c] + s[1][c];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        *reinterpret_cast<float2*>(part + (w * LONG_RUN + 4 * q + e) * KEPT + 2 * l) = make_float2(y[0][e], y[1][e]);
    __syncthreads();
    const int no = n0 + 2 * s32;
    if (live && s32 < KEPT / 2 && no < D) {
        const float* s = part + j * KEPT + 2 * s32;
        floatx2 v[PT / 64];
#pragma unroll
        for (int k = 0; k < PT / 64; ++k) v[k] = *reinterpret_cast<const floatx2*>(s + k * LONG_RUN * KEPT);
#pragma unroll
        for (int d = PT / 128; d > 0; d /= 2)
#pragma unroll
            for (int k = 0; k < d; ++k) v[k] += v[k + d];
        *reinterpret_cast<floatx2*>(r.Gent + (HEAD ? r.b + i : i) * D + no) = v[0];
        if (!UPDATE) *reinterpret_cast<float2*>((HEAD ? r.GU : r.GW) + i * D + no) = *reinterpret_cast<const float2*>(go + j * GP + no);
    }
    if (!UPDATE) return;

    float2 kf[LONG_RUN / 4];
#pragma unroll
    for (int k = 0; k < LONG_RUN / 4; ++k) kf[k] = *reinterpret_cast<const float2*>(ke + (4 * k + q) * KEPT + 2 * l);
#pragma unroll
    for (int t = 0; t < RUN_TILES; ++t) {
        if (t >= per) break;
        const int x = x0 + 16 * t + 4 * q, xa = x0 + 16 * t + l;
        floatx4 g[2] = {};
#pragma unroll
        for (int k = 0; k < LONG_RUN / 4; ++k) {
            if (4 * k >= m) break;
            const float f = go[(4 * k + q) * GP + xa];  // (xa < 256)
            g[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(f, kf[k].x, g[0], 0, 0, 0);
            g[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(f, kf[k].y, g[1], 0, 0, 0);
        }
        if (x >= D || n >= D) continue;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) M[t].v[c][e] -= adagrad1(g[c][e], S[t].v[c][e], a.lr, a.eps);
        if (HEAD) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t off = 4 * ((x + e) * D + n);
                const floatx2 v = {S[t].v[0][e], S[t].v[1][e]};
                if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<floatx2*>(to(St, off)));
                else *reinterpret_cast<floatx2*>(to(St, off)) = v;
                *reinterpret_cast<float2*>(to(T, off)) = make_float2(M[t].v[0][e], M[t].v[1][e]);
            }
        } else {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint32_t off = 4 * ((n + c) * D + x);
                st4(to(St, off), make_float4(S[t].v[c][0], S[t].v[c][1], S[t].v[c][2], S[t].v[c][3]));
                st4(to(T, off), make_float4(M[t].v[c][0], M[t].v[c][1], M[t].v[c][2], M[t].v[c][3]));
            }
        }
    }
}

template <bool UPDATE, bool STREAM, class Ids>
__device__ __forceinline__ void rescal_run_part(const RescalUpdArgs& a, int side, Ids ids_of, uint32_t key, int m, int slab, float* lds) {
    if (side == KGE_NEG_HEAD) rescal_run_part<true, UPDATE, STREAM>(a, ids_of, key, m, slab, lds);
    else rescal_run_part<false, UPDATE, STREAM>(a, ids_of, key, m, slab, lds);
}

// The runs of equal keys, in sorted order, long and short ones in lists of their own.
constexpr int LIST = 4096;
static_assert(1 + LIST + LONG_RUN + 2 * PT / 64 <= RUNS_LDS, "keys in LDS");
__device__ __forceinline__ void list_runs(const uint32_t* key, int n, RescalRuns* out, float* lds) {
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    uint32_t* const k = (uint32_t*)lds + 1;  // the keys from t0 - 1 on
    int* const sums = (int*)(k + LIST + LONG_RUN);
    RescalRun* const at[2] = {(RescalRun*)(out + 1), (RescalRun*)(out + 1) + n};
    int count[2] = {0, 0};
    for (int t0 = 0; t0 < n; t0 += LIST) {
        const int here = min(LIST, n - t0), halo = min(here + LONG_RUN, n - t0);
        __syncthreads();
        for (int e = tid - 1; e < halo; e += PT) k[e] = key[t0 + e < 0 ? 0 : t0 + e];
        __syncthreads();
        for (int e0 = 0; e0 < here; e0 += PT) {
            const int e = e0 + tid;
            const bool begins = e < here && (t0 + e == 0 || k[e - 1] != k[e]);
            int len = 1;  // of a short run (a long one's end is looked for where it is used)
#pragma unroll
            for (int x = 1; x < LONG_RUN; ++x) len += e + x < halo && k[e + x < halo ? e + x : 0] == k[e < halo ? e : 0];
            const bool is_long = begins && len == LONG_RUN;
            const unsigned long long bal[2] = {__ballot(begins && !is_long), __ballot(is_long)};
            __syncthreads();
            if (lane < 2) sums[2 * w + lane] = __popcll(bal[lane]);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                int before = count[s] + __popcll(bal[s] & ((1ull << lane) - 1));
                for (int v = 0; v < PT / 64; ++v) {
                    if (v < w) before += sums[2 * v + s];
                    count[s] += sums[2 * v + s];
                }
                if (begins && is_long == (s == 1)) at[s][before] = {k[e], t0 + e, len};
            }
        }
    }
    if (tid < 2) out->count[tid] = count[tid];
}

// The chain rule of the long runs: workgroups of (16 sorted positions, first or second long run among them, slab), behind one that lists the
// runs for the launch after this.  Few and short for steps of few relations, whose time is that of one workgroup: key -> position -> ids -> rows.
// Positions are asked for beside the keys, and a second run does not wait for the first.  us per step, head corrupted, the chain rule
// per positive -> one workgroup for both runs, positions after the keys -> this (b, k, D, relations):  76, 16, 160, 3 37.8 -> 41.1 -> 37.6;  312, 240, 148, 3
// 42.6 -> 44.7 -> 41.1;  512, 64, 200, 3 49.2 -> 49.6 -> 47.7;  1024, 256, 256, 3 80.6 -> 69.5 -> 68.8.
__global__ __launch_bounds__(PT) void k_rescal_chain_runs(RescalUpdArgs a) {
    __shared__ __attribute__((aligned(16))) float lds[RUNS_LDS];
    const int slabs = (a.D + KEPT - 1) / KEPT, wg = flat_block() - 1;
    if (wg < 0) {
        list_runs(a.key, a.n, a.runs, lds);
        return;
    }
    const int blocks = (a.n + LONG_RUN - 1) / LONG_RUN, b0 = wg / slabs % blocks * LONG_RUN, slab = wg % slabs;
    int others = wg / slabs / blocks;  // long runs that come before this workgroup's
    if (others > 1) return;
    // lane t: position b0 + t - 16, those of the 16 and 16 on either side
    const int lane = threadIdx.x & 63, e = b0 + lane - LONG_RUN;
    const bool in = e >= 0 && e < a.n && lane < 3 * LONG_RUN;
    const uint32_t mine = a.key[in ? e : 0];
    const uint32_t pos = a.pos[min(b0 + (lane & (LONG_RUN - 1)), a.n - 1)];  // lane t: of b0 + t
    const StepView sv = step_view(a.chain.ids);
    for (int s = 0; s < LONG_RUN && b0 + s < a.n;) {
        const uint32_t key = __builtin_amdgcn_readlane(mine, LONG_RUN + s);
        const unsigned long long eq = __ballot(in && mine == key);
        const int m = __builtin_ctzll(~(eq >> (LONG_RUN + s))), here = min(m, LONG_RUN - s);
        if (__popcll(eq) >= LONG_RUN && others-- == 0) {
            // (ahead of the matrix, which what waits for them would wait for too)
            const uint32_t hid = (uint32_t)clamp_id(sv.h[pos], a.chain.n_ent), tl = (uint32_t)clamp_id(sv.t[pos], a.chain.n_ent);
            const float cp = a.chain.cpos[pos];
            rescal_run_part<false, false>(a, sv.side, [&](int j, int m, int64_t& i, int64_t& h, int64_t& t, float& c) {
                const int from = s + min(j + (lane >> 5), m - 1);
                i = __shfl((int)pos, from, 64); h = (uint32_t)__shfl((int)hid, from, 64); t = (uint32_t)__shfl((int)tl, from, 64); c = __shfl(cp, from, 64);
            }, key, here, slab, lds);
            return;
        }
        s += here;
    }
}

// Rows of 148 to 256 floats.  us per FB15k-sized training step, b 1024, chain rule per positive and update by slabs -> by runs:
// D 200 119.9 -> 112.6 (100 relations 80.2 -> 65.0, 10 68.6 -> 61.4), 256 167 -> 143, 148 tail 81.0 -> 72.6, head 76.9 -> 75.0.  Shorter
// rows gain with the tail corrupted (132 70.2 -> 65.5, 100 57.0 -> 54.7) and lose with the head (144 72.2 -> 72.9, 132 68.0 -> 71.1, 100
// 55.4 -> 58.5): the columns of a workgroup start and end inside of cache lines.  For the same reason the state is stored past the
// caches there (STREAM) where the tables are far beyond them (D 200 116.2 -> 112.8, 180 102.8 -> 99.7; 275 MB of tables, D 160,
// 79.0 -> 81.6).
// Workgroups: the tiles of the long runs, then 8 * slabs for every 8 short runs: the slabs of a run are workgroups of one XCD,
// whose L2 then holds the lines that two of them share.
template <bool STREAM>  // matrices and state are more than what the Infinity Cache holds, and a quarter
__global__ __launch_bounds__(PT, 6) void k_rescal_runs(RescalUpdArgs a) {
    __shared__ __attribute__((aligned(16))) float lds[RUNS_LDS];
    __shared__ int first_other;
    const int tiles = (a.D + LT - 1) / LT, slabs = (a.D + KEPT - 1) / KEPT;
    const RescalRun* list = (const RescalRun*)(a.runs + 1);
    const int block = flat_block(), long_wgs = a.runs->count[1] * tiles * tiles;
    if (block < long_wgs) {
        const int q = block / (tiles * tiles);
        const RescalRun run = list[a.n + q];
        rescal_long_run<PT>(a, run.key, run.first, block - q * tiles * tiles, tiles, lds, (uint32_t*)(lds + PT / 64 * LT * LT), &first_other);
        return;
    }
    const int wg = block - long_wgs, eight = wg / (8 * slabs), in = wg - eight * 8 * slabs;
    const int q = 8 * eight + (in & 7), slab = in >> 3;
    if (q >= a.runs->count[0]) return;
    const RescalRun run = list[q];
    const StepView sv = step_view(a.chain.ids);
    rescal_run_part<true, STREAM>(a, sv.side, [&](int j, int m, int64_t& i, int64_t& h, int64_t& t, float& c) {
        // (the same for the whole wave: scalar loads, which do not wait for the matrix)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t iu = __builtin_amdgcn_readfirstlane(a.pos[run.first + min(j + u, m - 1)]);
            const int64_t hu = clamp_id(sv.h[iu], a.chain.n_ent), tu = clamp_id(sv.t[iu], a.chain.n_ent);
            const float cu = a.chain.cpos[iu];
            const bool mine = (threadIdx.x >> 5 & 1) == u;
            i = mine ? iu : i; h = mine ? hu : h; t = mine ? tu : t; c = mine ? cu : c;
        }
    }, run.key, run.n, slab, lds);
}

RescalArgs make_args(kge_ctx* c, const float* E, const float* R, const StepIds& ids) {
    RescalArgs a = {};
    a.E = E; a.R = R; a.ids = ids; a.b = ids.b; a.D = c->cfg.ent_dim;
    a.n_ent = c->cfg.num_entities; a.n_rel = c->cfg.num_relations;
    a.O = c->O; a.GO = c->GO; a.cpos = c->cpos; a.Gent = c->Gent;
    a.GU = c->Grel; a.GW = c->Grel + (int64_t)ids.b * c->cfg.ent_dim;  // the relation-gradient area holds the factors
    return a;
}

}  // namespace

void kge_launch_rescal_phi(kge_ctx* c, const float* E, const float* R, const StepIds& ids, hipStream_t st) {
    const RescalArgs a = make_args(c, E, R, ids);
    if (a.D > 256) KGE_LAUNCH(c, (k_rescal<false, true>), dim3(a.b), dim3(RT), 0, st, a);
    else KGE_LAUNCH(c, (k_rescal<false, false>), dim3(a.b), dim3(RT), 0, st, a);
}

size_t kge_rescal_runs_bytes(const kge_config& cfg) { return sizeof(RescalRuns) + 2 * sizeof(RescalRun) * (size_t)cfg.max_batch; }

bool kge_rescal_chain_by_runs(const kge_ctx* c) { return c->cfg.ent_dim >= RUNS_MIN_D && c->cfg.ent_dim <= RUNS_D; }

namespace {
RescalUpdArgs make_update_args(kge_ctx* c, const float* E, float* R, float* SR, const StepIds& ids, float lr) {
    RescalUpdArgs a;
    const int D = c->cfg.ent_dim;
    int rows = 1024 / D;  // matrix rows per workgroup: the largest divisor of D that keeps a slab within 1024 floats
    while (D % rows != 0) --rows;
    a.T = R; a.St = SR; a.key = c->rkey[c->rbuf]; a.pos = c->rpos[c->rbuf];
    a.n = ids.b; a.D = D; a.rows_per_slab = rows; a.long_y = 0;
    a.GU = c->Grel; a.GW = c->Grel + (int64_t)ids.b * D;
    a.lr = lr; a.eps = c->eps;
    a.chain = make_args(c, E, R, ids);
    a.runs = (RescalRuns*)c->rescal_runs;
    return a;
}
}  // namespace

void kge_launch_rescal_chain(kge_ctx* c, const float* E, float* R, const StepIds& ids, bool ordered, hipStream_t st) {
    if (kge_rescal_chain_by_runs(c)) {
        const int64_t slabs = (c->cfg.ent_dim + KEPT - 1) / KEPT;
        KGE_LAUNCH(c, k_rescal_chain_runs, flat_grid(1 + (ids.b + LONG_RUN - 1) / LONG_RUN * 2 * slabs), dim3(PT), 0, st,
                   make_update_args(c, E, R, nullptr, ids, 0.f));
        return;
    }
    RescalArgs a = make_args(c, E, R, ids);
    if (ordered) { a.key = c->rkey[c->rbuf]; a.pos = c->rpos[c->rbuf]; }
    const dim3 grid(a.pos ? (a.b + 7) / 8 * 8 : a.b);
    if (a.D > 256) KGE_LAUNCH(c, (k_rescal<true, true>), grid, dim3(RT), 0, st, a);
    else KGE_LAUNCH(c, (k_rescal<true, false>), grid, dim3(RT), 0, st, a);
}

void kge_launch_rescal_update(kge_ctx* c, const float* E, float* R, float* SR, const StepIds& ids, float lr, hipStream_t st) {
    RescalUpdArgs a = make_update_args(c, E, R, SR, ids, lr);
    const int tiles = (a.D + LT - 1) / LT;
    if (kge_rescal_chain_by_runs(c)) {
        // most workgroups where all runs are short: a long one has tiles * tiles <= LONG_RUN * slabs
        const int64_t slabs = (a.D + KEPT - 1) / KEPT;
        static_assert(LT == KEPT && RUNS_D / LT <= LONG_RUN);
        const dim3 grid = flat_grid((ids.b + 7) * slabs);
        const bool stream = (int64_t)c->cfg.num_relations * a.D * a.D * 8 > (int64_t)320 << 20;
        if (stream) KGE_LAUNCH(c, k_rescal_runs<true>, grid, dim3(PT), 0, st, a);
        else KGE_LAUNCH(c, k_rescal_runs<false>, grid, dim3(PT), 0, st, a);
        return;
    }
    const int64_t long_wgs = ids.b < LONG_RUN ? 0 : (int64_t)((ids.b + LONG_RUN - 1) / LONG_RUN) * tiles * tiles;
    a.long_y = (int)((long_wgs + ids.b - 1) / ids.b);
    KGE_LAUNCH(c, k_rescal_update, dim3(ids.b, a.long_y + a.D / a.rows_per_slab), dim3(RT), 0, st, a);
}
