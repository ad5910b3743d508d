// Chunks of ONE positive: every positive has corrupting entities of its own (the sampling that Sec. 3.3 of the paper
// compares joint sampling with).  No corrupting row is shared, so there is no matrix product to form: a 32-row
// tile would hold one real row.  The work is to read b * k rows once, and this kernel does everything that needs
// them in that one pass: a workgroup per positive forms o = phi(a, r), scores the positive and its k negatives, turns
// every score into its coefficient W = dL/df-, adds the negative to dL/do while its row is still in registers, and
// ends with the chain rule to the positive's three gradient rows.  The corrupting rows' own gradients W_j dir(o, n_j) are
// never stored: what is left behind is W and o, and k_update_runs forms each term while it adds up the row.
//
// Bound by the rows that travel from the Infinity Cache or memory (1600 bytes each at D = 400).  SUB lanes share a row
// (16 or 32 for short rows, so that a wave works on several), four rows per lane group are in flight while the four
// before them are worked on, and the four scores are reduced together (each halving step hands half of the rows
// to the other lanes: 7 shuffles instead of 24).  Weights that need all scores of a positive (self-adversarial softmax)
// are formed on line: running maximum, rescaled sums.  b = 1024, k = 256, D = 400, TransE-L2 on the FB15k-sized graph: 60 us
// = 420 MB of rows at 7 TB/s, where gather, forward and backward products took 128 + 111 + 604 us.
#include "k_gemm_shared.h"
#include "k_weights.h"

namespace {

constexpr int IT = 256;  // threads per workgroup
constexpr int U = 4;     // rows per lane group and round

enum { IND_SCORE = 0, IND_UNIFORM = 1, IND_GENERAL = 2 };

struct IndArgs {
    const float* E;
    const float* R;
    StepIds ids;
    int b, k, D, Dr;
    int64_t n_ent, n_rel;
    float gamma, alpha, wk;  // wk = 1 / (k b)
    int ranking;
    float* O;         // [b x D]
    float* S;         // IND_SCORE: scores (may be null: positives only); else W
    int ld_s;
    float* fpos;
    float* pos_out;
    float* cpos;
    float* row_loss;
    float* Gent;
    float* Grel;
};

template <int SUB> __device__ __forceinline__ float sub_sum(float v) {
#pragma unroll
    for (int o = SUB / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sums of four values over SUB lanes at once; lane group q (of SUB / 4 lanes) of the SUB ends with the sum of value q.
template <int SUB> __device__ __forceinline__ float sub_sum4(const float (&s)[U], int ln) {
    const bool h1 = ln & (SUB / 2), h2 = ln & (SUB / 4);
    float a = h1 ? s[2] : s[0], b = h1 ? s[3] : s[1];
    a += __shfl_xor(h1 ? s[0] : s[2], SUB / 2, 64);
    b += __shfl_xor(h1 ? s[1] : s[3], SUB / 2, 64);
    float c = h2 ? b : a;
    c += __shfl_xor(h2 ? a : b, SUB / 4, 64);
#pragma unroll
    for (int o = SUB / 8; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    return c;
}
// value q of sub_sum4's result, for all SUB lanes
template <int SUB> __device__ __forceinline__ float sub_pick(float v, int q, int lane) {
    if (SUB == 64) return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), q * 16));
    return __shfl(v, (lane & ~(SUB - 1)) + q * (SUB / 4), 64);
}

// MODE: IND_SCORE forward only; IND_UNIFORM logistic loss with weights 1/k; IND_GENERAL softmax weights and / or the
// ranking loss.  A row is NV 16-byte pieces per lane (complex models: NV pairs of a real and an imaginary piece).
// LONG: more than KGE_SHORT_SCORES corrupting rows per positive.
template <int MODEL, int SUB, int NV, int MODE, bool BF, bool LONG>
__global__ __launch_bounds__(IT) void k_ind(IndArgs a) {
    constexpr bool CPLX = MODEL == KGE_COMPLEX || MODEL == KGE_ROTATE;
    constexpr bool DOT = MODEL == KGE_DISTMULT || MODEL == KGE_COMPLEX;
    constexpr int NP = CPLX ? 2 * NV : NV;  // 16-byte pieces per lane
    constexpr int NS = IT / SUB;            // lane groups per workgroup
    constexpr bool TRAIN = MODE != IND_SCORE;
    __shared__ __attribute__((aligned(16))) float4 part[TRAIN ? NS - 1 : 1][TRAIN ? SUB * NP : 1];
    __shared__ float s_m[NS], s_z[NS], s_l[NS], s_act[NS];
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, ln = tid & (SUB - 1), sub = tid / SUB;
    const int D = a.D, k = a.k, nvec = CPLX ? D / 8 : D / 4, im_off = D / 2;
    const StepView sv = step_view(a.ids);
    const bool head = sv.side == KGE_NEG_HEAD;
    const int64_t hid = clamp_id(sv.h[i], a.n_ent), tl = clamp_id(sv.t[i], a.n_ent), rid = clamp_id(sv.r[i], a.n_rel);
    const float* pa = a.E + (head ? tl : hid) * (int64_t)D;
    const float* pc = a.E + (head ? hid : tl) * (int64_t)D;
    const float* pr = a.R + rid * (int64_t)a.Dr;
    const int64_t* neg = sv.neg + (int64_t)i * k;

    bool ok[NV];
    int off[NP];
#pragma unroll
    for (int it = 0; it < NV; ++it) {
        const int v = ln + it * SUB;
        ok[it] = v < nvec;
        const int o4 = 4 * (ok[it] ? v : 0);  // lanes past the row's end read its first piece; what they form is left out
        if (CPLX) { off[2 * it] = o4; off[2 * it + 1] = im_off + o4; }
        else off[it] = o4;
    }

    // rows of the round after next are asked for by id one round earlier
    const int per_round = NS * U;
    const int rounds = a.S ? (k + per_round - 1) / per_round : 0;
    auto row_id = [&](int rd, int u) {
        const int j = rd * per_round + sub * U + u;
        return clamp_id(neg[j < k ? j : k - 1], a.n_ent);
    };
    int64_t nid[U];
    float4 nx[U][NP];
    if (rounds > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) nid[u] = row_id(0, u);
    }

    // ---- o and the positive's score
    float o[4 * NP], oq[4 * NP];  // oq: as the products see it (rounded with bf16 operands)
    float fp;
    {
        float4 Av[NP], Cv[NP], Rv[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            Av[p] = ld4(pa + off[p]);
            Cv[p] = ld4(pc + off[p]);
            if (MODEL != KGE_ROTATE) Rv[p] = ld4(pr + off[p]);
            else if ((p & 1) == 0) Rv[p] = ld4(pr + off[p]);
        }
        float acc = 0.f;
#pragma unroll
        for (int it = 0; it < NV; ++it) {
            float s = 0.f;
            if constexpr (!CPLX) {
                const float av[4] = {Av[it].x, Av[it].y, Av[it].z, Av[it].w}, rv[4] = {Rv[it].x, Rv[it].y, Rv[it].z, Rv[it].w};
                const float cv[4] = {Cv[it].x, Cv[it].y, Cv[it].z, Cv[it].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float ov = MODEL == KGE_DISTMULT ? av[e] * rv[e] : (head ? av[e] - rv[e] : av[e] + rv[e]);
                    o[4 * it + e] = ov;
                    const float q = ov - cv[e];
                    s += MODEL == KGE_DISTMULT ? ov * cv[e] : (MODEL == KGE_TRANSE_L1 ? fabsf(q) : q * q);
                }
            } else {
                const float4 Ar = Av[2 * it], Ai = Av[2 * it + 1], Cr = Cv[2 * it], Ci = Cv[2 * it + 1], R0 = Rv[2 * it];
                const float are[4] = {Ar.x, Ar.y, Ar.z, Ar.w}, aim[4] = {Ai.x, Ai.y, Ai.z, Ai.w};
                const float cre[4] = {Cr.x, Cr.y, Cr.z, Cr.w}, cim[4] = {Ci.x, Ci.y, Ci.z, Ci.w};
                float rre[4] = {R0.x, R0.y, R0.z, R0.w}, rim[4];
                if (MODEL == KGE_ROTATE) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) { const float th = rre[e]; sincosf(th, &rim[e], &rre[e]); }
                } else {
                    const float4 R1 = Rv[2 * it + 1];
                    rim[0] = R1.x; rim[1] = R1.y; rim[2] = R1.z; rim[3] = R1.w;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float ri = head ? -rim[e] : rim[e];
                    const float ore = are[e] * rre[e] - aim[e] * ri, oim = are[e] * ri + aim[e] * rre[e];
                    o[8 * it + e] = ore;
                    o[8 * it + 4 + e] = oim;
                    if (MODEL == KGE_COMPLEX) s += ore * cre[e] + oim * cim[e];
                    else { const float qr = ore - cre[e], qi = oim - cim[e]; s += sqrtf(qr * qr + qi * qi); }
                }
            }
            acc += ok[it] ? s : 0.f;
        }
        acc = sub_sum<SUB>(acc);
        fp = MODEL == KGE_TRANSE_L2 ? a.gamma - sqrtf(acc) : (DOT ? acc : a.gamma - acc);
#pragma unroll
        for (int e = 0; e < 4 * NP; ++e) oq[e] = BF ? round_bf16(o[e]) : o[e];
    }

    if (rounds > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int p = 0; p < NP; ++p) nx[u][p] = ld4(a.E + nid[u] * (int64_t)D + off[p]);
        }
        if (rounds > 1) {
#pragma unroll
            for (int u = 0; u < U; ++u) nid[u] = row_id(1, u);
        }
    }
    float go[4 * NP];
#pragma unroll
    for (int e = 0; e < 4 * NP; ++e) go[e] = 0.f;
    float m = -INFINITY, z = 0.f, li = 0.f, active = 0.f;  // IND_GENERAL: running maximum, sums scaled by exp(-m)
    const bool owner = (ln & (SUB / 4 - 1)) == 0;          // one lane per row counts its loss and stores its value
    float* Srow = a.S + (int64_t)i * a.ld_s;
    for (int rd = 0; rd < rounds; ++rd) {
        float q[U][4 * NP];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                q[u][4 * p] = nx[u][p].x; q[u][4 * p + 1] = nx[u][p].y; q[u][4 * p + 2] = nx[u][p].z; q[u][4 * p + 3] = nx[u][p].w;
            }
        }
        if (rd + 1 < rounds) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int p = 0; p < NP; ++p) nx[u][p] = ld4(a.E + nid[u] * (int64_t)D + off[p]);
            }
            if (rd + 2 < rounds) {
#pragma unroll
                for (int u = 0; u < U; ++u) nid[u] = row_id(rd + 2, u);
            }
        }
        // q becomes the direction of dL/do per unit of W: n for the products, n - o for TransE-L2 (W carries the
        // 1 / distance), the negated sign or unit vector for the elementwise models
        float s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            s[u] = 0.f;
#pragma unroll
            for (int it = 0; it < NV; ++it) {
                float t = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (MODEL == KGE_ROTATE) {
                        const float qr = q[u][8 * it + e] - o[8 * it + e], qi = q[u][8 * it + 4 + e] - o[8 * it + 4 + e];
                        const float m2 = fmaf(qi, qi, qr * qr);
                        // (the modulus from the square root itself: m2 * rsq(m2) is an ulp worse, the same way in every
                        // coordinate); m2 = 0 gives 0 times a finite factor in the direction
                        const float rs = __builtin_amdgcn_rsqf(fmaxf(m2, 1.2e-38f));
                        t += __builtin_amdgcn_sqrtf(m2);
                        q[u][8 * it + e] = qr * rs;
                        q[u][8 * it + 4 + e] = qi * rs;
                    } else if constexpr (CPLX) {
                        if (BF) { q[u][8 * it + e] = round_bf16(q[u][8 * it + e]); q[u][8 * it + 4 + e] = round_bf16(q[u][8 * it + 4 + e]); }
                        t += q[u][8 * it + e] * oq[8 * it + e] + q[u][8 * it + 4 + e] * oq[8 * it + 4 + e];
                    } else {
                        float& x = q[u][4 * it + e];
                        if (BF) x = round_bf16(x);
                        if (MODEL == KGE_DISTMULT) t += x * oq[4 * it + e];
                        else {
                            x -= oq[4 * it + e];
                            t += MODEL == KGE_TRANSE_L1 ? fabsf(x) : x * x;
                        }
                    }
                }
                s[u] += ok[it] ? t : 0.f;
            }
        }
        const float tot = sub_sum4<SUB>(s, ln);
        const int j = rd * per_round + sub * U + ln / (SUB / 4);
        const bool real = j < k;
        const float d = MODEL == KGE_TRANSE_L2 ? sqrtf(tot) : 0.f;
        const float f = MODEL == KGE_TRANSE_L2 ? a.gamma - d : (DOT ? tot : a.gamma - tot);
        if (MODE == IND_SCORE) {
            if (owner && real) Srow[j] = f;
            continue;
        }
        float w;
        if (MODE == IND_UNIFORM) {
            float l = 0.f;
            if (DOT || MODEL == KGE_TRANSE_L2) {  // as the products of larger chunks do for rows of any length
                w = w_and_loss<!BF>(f, a.wk, l);
            } else {
                float sg;
                softplus_sigmoid_of<LONG>(f, l, sg);
                w = a.wk * sg;
            }
            if (MODEL == KGE_TRANSE_L2) w = d > 0.f ? w * (BF ? rcp_refined(d) : __builtin_amdgcn_rcpf(d)) : 0.f;
            if (BF) w = round_bf16(w);
            if (!real) w = 0.f;
            if (owner && real) {
                li += l;
                Srow[j] = w;
            }
        } else {
            if (owner && real) Srow[j] = MODEL == KGE_TRANSE_L2 ? d : f;
            float e = real ? 1.f : 0.f;
            if (a.alpha > 0.f) {
                float mx = real ? a.alpha * f : -INFINITY;
                mx = fmaxf(mx, __shfl_xor(mx, SUB / 2, 64));
                mx = fmaxf(mx, __shfl_xor(mx, SUB / 4, 64));
                if (mx > m) {  // (the same in all lanes of the group)
                    const float r = softmax_exp<LONG>(m - mx);
                    z *= r; li *= r; active *= r;
#pragma unroll
                    for (int x = 0; x < 4 * NP; ++x) go[x] *= r;
                    m = mx;
                }
                // (m is still -inf where every score so far was, i.e. distances beyond the floats: weight 0)
                e = real && m > -INFINITY ? softmax_exp<LONG>(a.alpha * f - m) : 0.f;
            }
            if (a.ranking) {
                const float t = a.gamma - fp + f;
                w = t > 0.f ? e : 0.f;
                if (owner) { li += e * fmaxf(t, 0.f); active += w; z += e; }
            } else {
                float sp, sg;
                softplus_sigmoid_of<LONG>(f, sp, sg);
                w = e * sg;
                if (owner) { li += e * sp; z += e; }
            }
            if (MODEL == KGE_TRANSE_L2) w = d > 0.f ? w / d : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float wu = sub_pick<SUB>(w, u, lane);
#pragma unroll
            for (int e = 0; e < 4 * NP; ++e) {
                if (MODEL == KGE_TRANSE_L1) go[e] += q[u][e] > 0.f ? wu : (q[u][e] < 0.f ? -wu : 0.f);
                else go[e] = fmaf(wu, q[u][e], go[e]);
            }
        }
    }
    if (MODE == IND_SCORE) {
        if (tid == 0) {
            a.fpos[i] = fp;
            if (a.pos_out) a.pos_out[i] = fp;
        }
        return;
    }

    // ---- the lane groups' sums meet in the first one, in group order
    li = sub_sum<SUB>(li);
    if (MODE == IND_GENERAL) { z = sub_sum<SUB>(z); active = sub_sum<SUB>(active); }
    if (ln == 0) { s_m[sub] = m; s_z[sub] = z; s_l[sub] = li; s_act[sub] = active; }
    if (sub > 0) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
            part[sub - 1][p * SUB + ln] = make_float4(go[4 * p], go[4 * p + 1], go[4 * p + 2], go[4 * p + 3]);
    }
    __syncthreads();
    float gm = -INFINITY, gz = 0.f, gl = 0.f, ga = 0.f;
    const bool soft = MODE == IND_GENERAL && a.alpha > 0.f;
    if (soft) {
        for (int q = 0; q < NS; ++q) gm = fmaxf(gm, s_m[q]);
    }
    for (int q = 0; q < NS; ++q) {
        const float r = soft ? softmax_exp<LONG>(s_m[q] - gm) : 1.f;
        gz += r * s_z[q]; gl += r * s_l[q]; ga += r * s_act[q];
    }
    const float invb = 1.f / (float)a.b;
    if (MODE == IND_GENERAL) {  // the values left in S become coefficients
        const float wz = invb / gz;
        for (int j = tid; j < k; j += IT) {
            const float raw = Srow[j];
            const float f = MODEL == KGE_TRANSE_L2 ? a.gamma - raw : raw;
            const float e = soft ? softmax_exp<LONG>(a.alpha * f - gm) : 1.f;
            float sp, sg, w;
            if (a.ranking) {
                w = a.gamma - fp + f > 0.f ? e * wz : 0.f;
            } else {
                softplus_sigmoid_of<LONG>(f, sp, sg);
                w = e * wz * sg;
            }
            if (MODEL == KGE_TRANSE_L2) w = raw > 0.f ? w / raw : 0.f;
            Srow[j] = w;
        }
    }
    if (sub > 0) return;
    const float scale = MODE == IND_GENERAL ? invb / gz : 1.f;
    if (soft) {
        const float r = softmax_exp<LONG>(m - gm);
#pragma unroll
        for (int e = 0; e < 4 * NP; ++e) go[e] *= r;
    }
    for (int q = 1; q < NS; ++q) {
        const float r = soft ? softmax_exp<LONG>(s_m[q] - gm) : 1.f;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const float4 v = part[q - 1][p * SUB + ln];
            go[4 * p] += r * v.x; go[4 * p + 1] += r * v.y; go[4 * p + 2] += r * v.z; go[4 * p + 3] += r * v.w;
        }
    }
    // ---- the positive's loss terms, then the chain rule
    const float ef = expf(-fabsf(fp));
    float cp = -((fp >= 0.f ? ef : 1.f) / (1.f + ef)) * invb;
    float loss = (fmaxf(-fp, 0.f) + log1pf(ef)) * invb;
    if (MODE == IND_UNIFORM) loss += gl * a.wk;
    else if (a.ranking) { loss = gl * scale; cp = -ga * scale; }
    else loss += gl * scale;
    if (tid == 0) {
        a.fpos[i] = fp;
        a.cpos[i] = cp;
        a.row_loss[i] = loss;
    }
    float inv = 0.f;
    if (MODEL == KGE_TRANSE_L2) {
        float ss = 0.f;
#pragma unroll
        for (int it = 0; it < NV; ++it) {
            const float4 C = ld4(pc + off[it]);
            const float u0 = o[4 * it] - C.x, u1 = o[4 * it + 1] - C.y, u2 = o[4 * it + 2] - C.z, u3 = o[4 * it + 3] - C.w;
            ss += ok[it] ? u0 * u0 + u1 * u1 + u2 * u2 + u3 * u3 : 0.f;
        }
        ss = sub_sum<SUB>(ss);
        inv = ss > 0.f ? 1.f / sqrtf(ss) : 0.f;
    }
    float* gA = a.Gent + (int64_t)(head ? a.b + i : i) * D;
    float* gC = a.Gent + (int64_t)(head ? i : a.b + i) * D;
    float* gR = a.Grel + (int64_t)i * a.Dr;
    float* po = a.O + (int64_t)i * D;
#pragma unroll
    for (int it = 0; it < NV; ++it) {
        if (!ok[it]) continue;
        if constexpr (!CPLX) {
            const float4 C = ld4(pc + off[it]);
            const float cv[4] = {C.x, C.y, C.z, C.w};
            float oa[4], oc[4], orl[4];
            if (MODEL == KGE_DISTMULT) {
                const float4 A = ld4(pa + off[it]), Rr = ld4(pr + off[it]);
                const float av[4] = {A.x, A.y, A.z, A.w}, rv[4] = {Rr.x, Rr.y, Rr.z, Rr.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = go[4 * it + e] * scale + cp * cv[e];
                    oc[e] = cp * o[4 * it + e];
                    oa[e] = g * rv[e];
                    orl[e] = g * av[e];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float u = o[4 * it + e] - cv[e];
                    const float dir = MODEL == KGE_TRANSE_L2 ? u * inv : (float)((u > 0.f) - (u < 0.f));
                    const float g = go[4 * it + e] * scale - cp * dir;
                    oc[e] = cp * dir;
                    oa[e] = g;
                    orl[e] = head ? -g : g;
                }
            }
            st4(gA + off[it], make_float4(oa[0], oa[1], oa[2], oa[3]));
            st4(gC + off[it], make_float4(oc[0], oc[1], oc[2], oc[3]));
            st4(gR + off[it], make_float4(orl[0], orl[1], orl[2], orl[3]));
            st4(po + off[it], make_float4(o[4 * it], o[4 * it + 1], o[4 * it + 2], o[4 * it + 3]));
        } else {
            const int f0 = off[2 * it], f1 = off[2 * it + 1];
            const float4 Ar = ld4(pa + f0), Ai = ld4(pa + f1), Cr = ld4(pc + f0), Ci = ld4(pc + f1), R0 = ld4(pr + f0);
            const float are[4] = {Ar.x, Ar.y, Ar.z, Ar.w}, aim[4] = {Ai.x, Ai.y, Ai.z, Ai.w};
            const float cre[4] = {Cr.x, Cr.y, Cr.z, Cr.w}, cim[4] = {Ci.x, Ci.y, Ci.z, Ci.w};
            float rre[4] = {R0.x, R0.y, R0.z, R0.w}, rim[4];
            if (MODEL == KGE_ROTATE) {
#pragma unroll
                for (int e = 0; e < 4; ++e) { const float th = rre[e]; sincosf(th, &rim[e], &rre[e]); }
            } else {
                const float4 R1 = ld4(pr + f1);
                rim[0] = R1.x; rim[1] = R1.y; rim[2] = R1.z; rim[3] = R1.w;
            }
            float oar[4], oai[4], ocr[4], oci[4], or0[4], or1[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float ore = o[8 * it + e], oim = o[8 * it + 4 + e];
                float gr = go[8 * it + e] * scale, gi = go[8 * it + 4 + e] * scale;
                if (MODEL == KGE_COMPLEX) {
                    gr += cp * cre[e]; gi += cp * cim[e];
                    ocr[e] = cp * ore; oci[e] = cp * oim;
                } else {
                    const float qr = ore - cre[e], qi = oim - cim[e], m2 = qr * qr + qi * qi;
                    const float im = m2 > 0.f ? 1.f / sqrtf(m2) : 0.f;
                    gr -= cp * qr * im; gi -= cp * qi * im;
                    ocr[e] = cp * qr * im; oci[e] = cp * qi * im;
                }
                const float ri = head ? -rim[e] : rim[e];
                oar[e] = gr * rre[e] + gi * ri;
                oai[e] = gi * rre[e] - gr * ri;
                if (MODEL == KGE_COMPLEX) {
                    const float d_ri = -gr * aim[e] + gi * are[e];
                    or0[e] = gr * are[e] + gi * aim[e];
                    or1[e] = head ? -d_ri : d_ri;
                } else {
                    const float d_th = -gr * oim + gi * ore;
                    or0[e] = head ? -d_th : d_th;
                }
            }
            st4(gA + f0, make_float4(oar[0], oar[1], oar[2], oar[3]));
            st4(gA + f1, make_float4(oai[0], oai[1], oai[2], oai[3]));
            st4(gC + f0, make_float4(ocr[0], ocr[1], ocr[2], ocr[3]));
            st4(gC + f1, make_float4(oci[0], oci[1], oci[2], oci[3]));
            st4(gR + f0, make_float4(or0[0], or0[1], or0[2], or0[3]));
            if (MODEL == KGE_COMPLEX) st4(gR + f1, make_float4(or1[0], or1[1], or1[2], or1[3]));
            st4(po + f0, make_float4(o[8 * it], o[8 * it + 1], o[8 * it + 2], o[8 * it + 3]));
            st4(po + f1, make_float4(o[8 * it + 4], o[8 * it + 5], o[8 * it + 6], o[8 * it + 7]));
        }
    }
}

template <int MODEL, int SUB, int NV>
void launch_mode(kge_ctx* c, const IndArgs& a, int mode, hipStream_t st) {
    constexpr bool HAS_BF = MODEL == KGE_TRANSE_L2 || MODEL == KGE_DISTMULT || MODEL == KGE_COMPLEX;
    const dim3 grid(a.b), block(IT);
    constexpr bool PAIR = !HAS_BF;
    const bool lng = a.k > KGE_SHORT_SCORES;
    if (mode == IND_SCORE) KGE_LAUNCH(c, (k_ind<MODEL, SUB, NV, IND_SCORE, false, false>), grid, block, 0, st, a);
    else if (mode == IND_GENERAL && lng) KGE_LAUNCH(c, (k_ind<MODEL, SUB, NV, IND_GENERAL, false, true>), grid, block, 0, st, a);
    else if (mode == IND_GENERAL) KGE_LAUNCH(c, (k_ind<MODEL, SUB, NV, IND_GENERAL, false, false>), grid, block, 0, st, a);
    else if (HAS_BF && c->cfg.gemm_input == 1) KGE_LAUNCH(c, (k_ind<MODEL, SUB, NV, IND_UNIFORM, HAS_BF, false>), grid, block, 0, st, a);
    else if (PAIR && lng) KGE_LAUNCH(c, (k_ind<MODEL, SUB, NV, IND_UNIFORM, false, PAIR>), grid, block, 0, st, a);
    else KGE_LAUNCH(c, (k_ind<MODEL, SUB, NV, IND_UNIFORM, false, false>), grid, block, 0, st, a);
}

template <int MODEL>
void launch_rows(kge_ctx* c, const IndArgs& a, int mode, hipStream_t st) {
    constexpr bool CPLX = MODEL == KGE_COMPLEX || MODEL == KGE_ROTATE;
    const int pieces = CPLX ? a.D / 8 : a.D / 4;  // at most 256 (complex models: 128)
    if (pieces <= 16) launch_mode<MODEL, 16, 1>(c, a, mode, st);
    else if (pieces <= 32) launch_mode<MODEL, 32, 1>(c, a, mode, st);
    else if (pieces <= 64) launch_mode<MODEL, 64, 1>(c, a, mode, st);
    else if (pieces <= 128) launch_mode<MODEL, 64, 2>(c, a, mode, st);
    else if constexpr (!CPLX) launch_mode<MODEL, 64, 4>(c, a, mode, st);
}

void launch(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, float gamma, float* out, int ld_out,
            float* pos_out, int mode, hipStream_t st) {
    IndArgs a;
    a.E = E; a.R = R; a.ids = ids; a.b = ids.b; a.k = k; a.D = c->cfg.ent_dim; a.Dr = c->cfg.rel_dim;
    a.n_ent = c->cfg.num_entities; a.n_rel = c->cfg.num_relations;
    a.gamma = gamma; a.alpha = c->cfg.adv_temperature; a.wk = k > 0 ? 1.f / ((float)k * (float)ids.b) : 0.f;
    a.ranking = c->cfg.loss == KGE_LOSS_RANKING;
    a.O = c->O; a.S = out; a.ld_s = ld_out; a.fpos = c->fpos; a.pos_out = pos_out; a.cpos = c->cpos;
    a.row_loss = c->row_loss; a.Gent = c->Gent; a.Grel = c->Grel;
    switch (c->cfg.model) {
    case KGE_TRANSE_L2: launch_rows<KGE_TRANSE_L2>(c, a, mode, st); break;
    case KGE_TRANSE_L1: launch_rows<KGE_TRANSE_L1>(c, a, mode, st); break;
    case KGE_DISTMULT: launch_rows<KGE_DISTMULT>(c, a, mode, st); break;
    case KGE_COMPLEX: launch_rows<KGE_COMPLEX>(c, a, mode, st); break;
    default: launch_rows<KGE_ROTATE>(c, a, mode, st); break;
    }
}

}  // namespace

// Chunks of one positive, one of the five models whose relation is a row of at most ent_dim floats.  (With bf16 operands
// the coefficients are rounded before they are multiplied, which needs the final weights in the one pass over the rows:
// uniform weights only.)
bool kge_ind_step_fits(const kge_ctx* c, int g) {
    const bool rows = c->cfg.model != KGE_RESCAL && c->cfg.model != KGE_TRANSR;
    return g == 1 && rows && (c->cfg.gemm_input == 0 || kge_gemm_backward_forms_w(c));
}
bool kge_ind_score_fits(const kge_ctx* c, int g) {
    return g == 1 && c->cfg.model != KGE_RESCAL && c->cfg.model != KGE_TRANSR && c->cfg.gemm_input == 0;
}
void kge_ind_step(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, float gamma, hipStream_t st) {
    launch(c, E, R, ids, k, gamma, c->S, c->ld_s, nullptr, kge_gemm_backward_forms_w(c) ? IND_UNIFORM : IND_GENERAL, st);
}
void kge_ind_score(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, float gamma, float* out,
                   int ld_out, float* pos_out, hipStream_t st) {
    launch(c, E, R, ids, k, gamma, out, ld_out, pos_out, IND_SCORE, st);
}
