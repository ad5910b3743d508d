// Duplicate reduction, part 2, fused with the optimizer, for steps whose corrupting rows were not shared (chunks of one
// positive, k_ind.hip): the entity key list is long (2b + b k keys), a row occurs many times in it, and the gradient
// rows of the corrupting entities do not exist in memory.  The gradient of corrupting entity n against positive i is
// W dir(o_i, n), a function of one coefficient, the row o_i (b rows, which every L2 holds) and the table row itself:
//     TransE-L2   W (o - n)  = W o - W n       DistMult, ComplEx   W o
//     TransE-L1   W sign(o - n)                RotatE              W (o - n) / |o - n| per coordinate
// so it is formed here, while the row's terms are added up, instead of being written and read back.
//
// The sorted key list is cut into tiles of `tile` positions; a lane group (one thread per 16 bytes of a row, rounded up
// to a power of two up to a wave, whole waves beyond) walks a tile in order with eight rows in flight.  A run of equal keys
// inside the tile is finished on the spot.  A run that crosses tile edges leaves one partial row per tile, and
// k_update_runs_join, whose lane group of the tile where such a run ENDS adds them up in tile order, applies Adagrad
// to it.  No atomics; every sum has a fixed order.  Replaces, for these steps, k_update, which reads a gradient row
// per key: b = 1024, k = 256, D = 400 on the FB15k-sized graph, TransE-L2 (264,192 keys, 14,951 rows), per step
//     gather + products + update with stored gradients   128 + 111 + 604 + 276 us
//     k_ind + k_update_runs + join                         60 + 43 + 13 us (1134 -> 154 us with the sort and the relations)
#include "kge_common.h"

namespace {

constexpr int RU = 8;          // rows in flight per lane group
constexpr int MAX_TILE = 64;   // positions per tile
constexpr int WG = 256;

struct RunArgs {
    float* T;
    float* St;
    const float* G;       // gradient rows of the positives' entities, by key position (< n_pos)
    const float* O;       // o rows
    const float* W;       // coefficients [b x ld_w]
    int ld_w, k, n_pos;
    const uint32_t* key;
    const uint32_t* pos;
    int n, D, tile, tiles;
    float lr, eps;
    float* part;          // partial rows [2 tiles x D]: 2t: run that began before tile t; 2t + 1: run that leaves it
    float* part_w;        // [2 tiles] sums of W that belong to them (TransE-L2)
};

template <int L> __device__ __forceinline__ float group_sum(float v, float* lds) {
    // sum over the lane group; groups of several waves are the whole workgroup
    const int w = L < 64 ? L : 64;
#pragma unroll
    for (int o = w / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (L <= 64) return v;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int q = 0; q < L / 64; ++q) t += lds[q];
    return t;
}

// Adagrad on one row whose summed gradient is acc (TransE-L2: still without its - wsum x); NQ pieces per lane.
template <int L, int NQ, bool L2, bool ROWWISE, bool BF>
__device__ __forceinline__ void finish_row(const RunArgs& a, uint32_t id, const int (&off)[NQ], bool act, float4 (&acc)[NQ],
                                           float wsum, float* lds) {
    float* trow = a.T + (int64_t)id * a.D;
    float4 x[NQ];
#pragma unroll
    for (int p = 0; p < NQ; ++p) x[p] = ld4(trow + off[p]);
    if (L2) {
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            float4 q = x[p];
            if (BF) q = make_float4(round_bf16(q.x), round_bf16(q.y), round_bf16(q.z), round_bf16(q.w));
            acc[p].x -= wsum * q.x; acc[p].y -= wsum * q.y; acc[p].z -= wsum * q.z; acc[p].w -= wsum * q.w;
        }
    }
    if (!ROWWISE) {
        float* srow = a.St + (int64_t)id * a.D;
        float4 s[NQ];
#pragma unroll
        for (int p = 0; p < NQ; ++p) s[p] = ld4(srow + off[p]);
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            adagrad4(acc[p], x[p], s[p], a.lr, a.eps);
            if (act) {
                st4(srow + off[p], s[p]);
                st4(trow + off[p], x[p]);
            }
        }
    } else {
        float ss = 0.f;
#pragma unroll
        for (int p = 0; p < NQ; ++p) ss += acc[p].x * acc[p].x + acc[p].y * acc[p].y + acc[p].z * acc[p].z + acc[p].w * acc[p].w;
        ss = group_sum<L>(act ? ss : 0.f, lds);
        const float S_new = a.St[id] + ss / (float)a.D;
        const float scale = a.lr * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(S_new) + a.eps);
        if (L > 64) __syncthreads();  // every wave has read the old accumulator
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            x[p].x -= scale * acc[p].x; x[p].y -= scale * acc[p].y; x[p].z -= scale * acc[p].z; x[p].w -= scale * acc[p].w;
            if (act) st4(trow + off[p], x[p]);
        }
        if (threadIdx.x % L == 0) a.St[id] = S_new;
    }
}

enum { TERM_DOT = 0, TERM_L2 = 1, TERM_L1 = 2, TERM_ROT = 3 };

// L: threads per lane group.  RotatE: a lane holds a real piece and the imaginary piece of the same coordinates.
template <int TERM, int L, bool ROWWISE, bool BF>
__global__ __launch_bounds__(L > 64 ? L : WG) void k_update_runs(RunArgs a) {
    constexpr int GROUPS = L > 64 ? 1 : WG / L, THREADS = L > 64 ? L : WG;
    constexpr int NQ = TERM == TERM_ROT ? 2 : 1;
    constexpr bool NEED_X = TERM == TERM_L1 || TERM == TERM_ROT;
    __shared__ uint32_t s_key[GROUPS * MAX_TILE + 2];
    __shared__ int s_row[GROUPS * MAX_TILE];   // >= 0: row of O; < 0: ~ row of G
    __shared__ float s_w[GROUPS * MAX_TILE];
    __shared__ float s_red[4];
    const int tid = threadIdx.x, grp = L > 64 ? 0 : tid / L, ln = L > 64 ? tid : tid % L;
    const int P = a.tile, base = blockIdx.x * GROUPS * P;
    // keys base - 1 .. base + GROUPS P, and what each position adds
    for (int e = tid; e < GROUPS * P + 2; e += THREADS) {
        const int q = base - 1 + e;
        s_key[e] = a.key[q < 0 ? 0 : (q < a.n ? q : a.n - 1)];
    }
    for (int e = tid; e < GROUPS * P; e += THREADS) {
        const int q = base + e < a.n ? base + e : a.n - 1;
        const int p = (int)a.pos[q];
        int row = ~p;
        float w = 1.f;
        if (p >= a.n_pos) {
            row = (p - a.n_pos) / a.k;
            w = a.W[(int64_t)row * a.ld_w + (p - a.n_pos - row * a.k)];
        }
        s_row[e] = row;
        s_w[e] = w;
    }
    __syncthreads();
    const int t = blockIdx.x * GROUPS + grp;
    const int p0 = t * P, cnt = min(P, a.n - p0);
    if (cnt <= 0) return;
    const uint32_t* key = s_key + 1 + grp * P;  // key[j]: sorted position p0 + j
    const int* row = s_row + grp * P;
    const float* wgt = s_w + grp * P;
    const int nq = TERM == TERM_ROT ? a.D / 8 : a.D / 4;
    const bool act = ln < nq;
    int off[NQ];
    off[0] = act ? 4 * ln : 0;
    if (TERM == TERM_ROT) off[NQ - 1] = off[0] + a.D / 2;
    const bool before = p0 > 0 && key[-1] == key[0];

    float4 acc[NQ];
#pragma unroll
    for (int p = 0; p < NQ; ++p) acc[p] = f4(0.f);
    float wsum = 0.f;
    bool open = before;  // the run being added up began before this tile
    for (int j0 = 0; j0 < cnt; j0 += RU) {
        float4 g[RU][NQ], x[NEED_X ? RU : 1][NQ];
        int rw[RU];
        float w[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int j = j0 + u < cnt ? j0 + u : cnt - 1;
            rw[u] = row[j];
            w[u] = wgt[j];
            const float* src = rw[u] >= 0 ? a.O + (int64_t)rw[u] * a.D : a.G + (int64_t)~rw[u] * a.D;
#pragma unroll
            for (int p = 0; p < NQ; ++p) g[u][p] = ld4(src + off[p]);
            if (NEED_X) {
#pragma unroll
                for (int p = 0; p < NQ; ++p) x[NEED_X ? u : 0][p] = ld4(a.T + (int64_t)key[j] * a.D + off[p]);
            }
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int j = j0 + u;
            if (j >= cnt) break;
            const bool neg = rw[u] >= 0;
            if (NEED_X && neg) {
                if (TERM == TERM_L1) {
                    const float4 q = g[u][0], y = x[NEED_X ? u : 0][0];
                    acc[0].x += q.x > y.x ? w[u] : (q.x < y.x ? -w[u] : 0.f);
                    acc[0].y += q.y > y.y ? w[u] : (q.y < y.y ? -w[u] : 0.f);
                    acc[0].z += q.z > y.z ? w[u] : (q.z < y.z ? -w[u] : 0.f);
                    acc[0].w += q.w > y.w ? w[u] : (q.w < y.w ? -w[u] : 0.f);
                } else {
                    const float4 r0 = g[u][0], r1 = g[u][NQ - 1], y0 = x[NEED_X ? u : 0][0], y1 = x[NEED_X ? u : 0][NQ - 1];
                    const float qr[4] = {r0.x - y0.x, r0.y - y0.y, r0.z - y0.z, r0.w - y0.w};
                    const float qi[4] = {r1.x - y1.x, r1.y - y1.y, r1.z - y1.z, r1.w - y1.w};
                    float f[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        f[e] = w[u] * __builtin_amdgcn_rsqf(fmaxf(fmaf(qi[e], qi[e], qr[e] * qr[e]), 1.2e-38f));
                    acc[0].x = fmaf(f[0], qr[0], acc[0].x); acc[NQ - 1].x = fmaf(f[0], qi[0], acc[NQ - 1].x);
                    acc[0].y = fmaf(f[1], qr[1], acc[0].y); acc[NQ - 1].y = fmaf(f[1], qi[1], acc[NQ - 1].y);
                    acc[0].z = fmaf(f[2], qr[2], acc[0].z); acc[NQ - 1].z = fmaf(f[2], qi[2], acc[NQ - 1].z);
                    acc[0].w = fmaf(f[3], qr[3], acc[0].w); acc[NQ - 1].w = fmaf(f[3], qi[3], acc[NQ - 1].w);
                }
            } else {
#pragma unroll
                for (int p = 0; p < NQ; ++p) {
                    float4 q = g[u][p];
                    if (BF && neg) q = make_float4(round_bf16(q.x), round_bf16(q.y), round_bf16(q.z), round_bf16(q.w));
                    acc[p].x = fmaf(w[u], q.x, acc[p].x); acc[p].y = fmaf(w[u], q.y, acc[p].y);
                    acc[p].z = fmaf(w[u], q.z, acc[p].z); acc[p].w = fmaf(w[u], q.w, acc[p].w);
                }
                if (TERM == TERM_L2 && neg) wsum += w[u];
            }
            const bool last = j == cnt - 1;
            const bool same_next = p0 + j + 1 < a.n && key[j + 1] == key[j];
            if (same_next && !last) continue;
            // the run ends here, or leaves the tile
            if (open || same_next) {
                const int64_t slot = 2 * (int64_t)t + (open ? 0 : 1);
                if (act) {
#pragma unroll
                    for (int p = 0; p < NQ; ++p) st4(a.part + slot * a.D + off[p], acc[p]);
                }
                if (TERM == TERM_L2 && ln == 0) a.part_w[slot] = wsum;
            } else {
                finish_row<L, NQ, TERM == TERM_L2, ROWWISE, BF>(a, key[j], off, act, acc, wsum, s_red);
            }
            open = false;
#pragma unroll
            for (int p = 0; p < NQ; ++p) acc[p] = f4(0.f);
            wsum = 0.f;
        }
    }
}

// Workgroup t: if a run that began before tile t ends in it, add up its partial rows (the tile where it began, the tiles
// it fills, this one) and apply Adagrad.  The lane groups take consecutive stretches of the partial rows (a hub entity of
// in-batch negatives fills hundreds of tiles) and their sums meet in LDS in order.
template <int L> struct JoinShape {
    static constexpr int THREADS = L < 64 ? 256 : (L == 64 ? 256 : 4 * L > 1024 ? 1024 : 4 * L);
    static constexpr int GROUPS = THREADS / L;
};
template <int TERM, int L, bool ROWWISE, bool BF>
__global__ __launch_bounds__(JoinShape<L>::THREADS) void k_update_runs_join(RunArgs a) {
    constexpr int GROUPS = JoinShape<L>::GROUPS;
    constexpr int NQ = TERM == TERM_ROT ? 2 : 1;
    constexpr int JU = 8;
    __shared__ __attribute__((aligned(16))) float4 s_acc[GROUPS][NQ][L];
    __shared__ float s_w[GROUPS], s_red[4];
    const int tid = threadIdx.x, grp = tid / L, ln = tid % L, lane = tid & 63;
    const int t = blockIdx.x + 1, P = a.tile, p0 = t * P;
    const int p1 = min(p0 + P, a.n);
    const uint32_t key = a.key[p0];
    if (a.key[p0 - 1] != key) return;
    if (p1 < a.n && a.key[p1 - 1] == key && a.key[p1] == key) return;  // it goes on
    // tiles t - 1, t - 2, ... that the run fills: those with the key also just before their first position
    int full = 0;
    for (;;) {
        const int q = t - 1 - full - lane;
        const unsigned long long bal = __ballot(!(q > 0 && a.key[q > 0 ? q * P - 1 : 0] == key));
        const int first = bal == 0 ? 64 : __builtin_ctzll(bal);
        full += first;
        if (first < 64) break;
    }
    const int nq = TERM == TERM_ROT ? a.D / 8 : a.D / 4;
    const bool act = ln < nq;
    int off[NQ];
    off[0] = act ? 4 * ln : 0;
    if (TERM == TERM_ROT) off[NQ - 1] = off[0] + a.D / 2;
    // partials in order: slot 2 (t - 1 - full) + 1, then 2 q for q = t - full .. t
    const int q0 = t - 1 - full, m = full + 2;
    const int j1 = (int)((int64_t)m * (grp + 1) / GROUPS);
    float4 acc[NQ];
#pragma unroll
    for (int p = 0; p < NQ; ++p) acc[p] = f4(0.f);
    float wsum = 0.f;
    for (int j0 = (int)((int64_t)m * grp / GROUPS); j0 < j1; j0 += JU) {
        float4 g[JU][NQ];
        float w[JU];
#pragma unroll
        for (int u = 0; u < JU; ++u) {
            const int j = j0 + u < j1 ? j0 + u : j0;
            const int64_t slot = 2 * (int64_t)(q0 + j) + (j == 0 ? 1 : 0);
#pragma unroll
            for (int p = 0; p < NQ; ++p) g[u][p] = ld4(a.part + slot * a.D + off[p]);
            w[u] = TERM == TERM_L2 ? a.part_w[slot] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < JU; ++u) {
            if (j0 + u >= j1) break;
#pragma unroll
            for (int p = 0; p < NQ; ++p) { acc[p].x += g[u][p].x; acc[p].y += g[u][p].y; acc[p].z += g[u][p].z; acc[p].w += g[u][p].w; }
            wsum += w[u];
        }
    }
#pragma unroll
    for (int p = 0; p < NQ; ++p) s_acc[grp][p][ln] = acc[p];
    if (ln == 0) s_w[grp] = wsum;
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g2 = 1; g2 < GROUPS; ++g2) {
#pragma unroll
        for (int p = 0; p < NQ; ++p) {
            const float4 v = s_acc[g2][p][ln];
            acc[p].x += v.x; acc[p].y += v.y; acc[p].z += v.z; acc[p].w += v.w;
        }
        wsum += s_w[g2];
    }
    finish_row<L, NQ, TERM == TERM_L2, ROWWISE, BF>(a, key, off, act, acc, wsum, s_red);
}

template <int TERM, int L, bool ROWWISE, bool BF>
void launch_both(kge_ctx* c, const RunArgs& a, hipStream_t st) {
    constexpr int GROUPS = L > 64 ? 1 : WG / L;
    const dim3 grid((a.tiles + GROUPS - 1) / GROUPS), block(L > 64 ? L : WG);
    KGE_LAUNCH(c, (k_update_runs<TERM, L, ROWWISE, BF>), grid, block, 0, st, a);
    if (a.tiles > 1)
        hipLaunchKernelGGL((k_update_runs_join<TERM, L, ROWWISE, BF>), dim3(a.tiles - 1), dim3(JoinShape<L>::THREADS), 0, st, a);
}

template <int TERM, bool ROWWISE, bool BF>
void launch_width(kge_ctx* c, const RunArgs& a, hipStream_t st) {
    const int nq = TERM == TERM_ROT ? a.D / 8 : a.D / 4;
    if (nq <= 16) launch_both<TERM, 16, ROWWISE, BF>(c, a, st);
    else if (nq <= 32) launch_both<TERM, 32, ROWWISE, BF>(c, a, st);
    else if (nq <= 64) launch_both<TERM, 64, ROWWISE, BF>(c, a, st);
    else if (nq <= 128) launch_both<TERM, 128, ROWWISE, BF>(c, a, st);
    else launch_both<TERM, 256, ROWWISE, BF>(c, a, st);
}

template <int TERM, bool HAS_BF>
void launch_term(kge_ctx* c, const RunArgs& a, hipStream_t st) {
    const bool bf = HAS_BF && c->cfg.gemm_input == 1;
    if (c->cfg.adagrad_mode == 1) {
        if (bf) launch_width<TERM, true, HAS_BF>(c, a, st);
        else launch_width<TERM, true, false>(c, a, st);
    } else {
        if (bf) launch_width<TERM, false, HAS_BF>(c, a, st);
        else launch_width<TERM, false, false>(c, a, st);
    }
}

}  // namespace

// Entity rows of a step that k_ind ran (chunks of one positive).
void kge_launch_update_runs(kge_ctx* c, float* E, float* SE, const StepIds& ids, int k, float lr, hipStream_t st) {
    RunArgs a;
    a.T = E; a.St = SE; a.G = c->Gent; a.O = c->O; a.W = c->S; a.ld_w = c->ld_s; a.k = k; a.n_pos = 2 * ids.b;
    a.key = c->ekey[c->ebuf]; a.pos = c->epos[c->ebuf];
    a.n = 2 * ids.b + ids.n_neg; a.D = c->cfg.ent_dim;
    // short lists are cut finer, so that there are enough tiles for the chip
    a.tile = 8;
    while (a.tile < MAX_TILE && a.n / a.tile > 8192) a.tile *= 2;
    a.tiles = (a.n + a.tile - 1) / a.tile;
    a.lr = lr; a.eps = c->eps;
    // partial rows: the area of the corrupting rows' gradients, which such a step does not form (at most n / 4 rows)
    a.part = c->Gent + (int64_t)2 * ids.b * a.D; a.part_w = c->run_part_w;
    switch (c->cfg.model) {
    case KGE_TRANSE_L2: launch_term<TERM_L2, true>(c, a, st); break;
    case KGE_TRANSE_L1: launch_term<TERM_L1, false>(c, a, st); break;
    case KGE_ROTATE: launch_term<TERM_ROT, false>(c, a, st); break;
    default: launch_term<TERM_DOT, true>(c, a, st); break;
    }
}
