// Chunked negative scoring for the models whose pair function is not a bilinear form:
//     RotatE      psi(o, n) = gamma - sum_c |o_c - n_c|      (complex modulus per coordinate)
//     TransE-L1   psi(o, n) = gamma - sum_d |o_d - n_d|
// Sec. 3.3's grouping still applies (g positives share k corrupting rows, so each staged row is reused g or k
// times), but the g*k*D pair terms are an elementwise reduction with a square root or an absolute value in
// it, so they run on the vector ALUs, not on the matrix units.
//
// Forward: a workgroup owns a 32x32 tile of (positive, negative) pairs and stages 32 coordinates of both sides in
// LDS at a time; a thread accumulates a 2x2 block of pairs and reads four coordinates of a row with one 16-byte
// LDS load, so one load serves eight pair terms.  The modulus uses the hardware square root (1 ulp).
// Backward: threads own coordinates instead of pairs, so the sums over j (for dL/do_i) and over i (for the gradient row of
// corrupting entity j) stay in registers.  Both sums are made of the same terms W_ij dir(o_i - n_j) with opposite signs,
// and a term costs a reciprocal square root, so it is formed once: a workgroup owns a tile of positives x a range of
// negatives, a thread keeps its coordinate of the tile's o rows and of their running sums in registers, walks the negatives
// that fall to its thread group, and adds every term to both sides.  What a workgroup can sum is partial (over its
// negatives for dL/do, over its positives for a corrupting row): the partial rows go to a scratch area and the chain launch
// (k_chain) adds them in a fixed order.  The launch also turns the scores into the coefficients W = dL/df- while it stages
// them (softmax weights, logistic or ranking loss), and one workgroup per tile of positives sums the loss: there is no loss
// kernel between the two launches.
// Nothing is accumulated with atomics.
#include "k_weights.h"

namespace {

constexpr int PT = 32;       // pair tile edge
constexpr int PCK = 32;      // coordinates staged per step
constexpr int PPITCH = 36;   // floats per staged row: 16-byte aligned rows

struct PairArgs {
    const float* O;    // [b x D]
    const float* Nst;  // [C*k x D]
    float* S;          // [b x ld_s] scores: out of the forward, into the backward
    int ld_s, g, k, D;
    float gamma;
};

template <bool CPLX>
__device__ __forceinline__ float pair_term(float o_re, float o_im, float n_re, float n_im) {
    const float q_re = o_re - n_re;
    if (!CPLX) return fabsf(q_re);
    const float q_im = o_im - n_im;
    return __builtin_amdgcn_sqrtf(q_re * q_re + q_im * q_im);
}

// 512 threads: both halves of the workgroup hold the same 2x2 blocks of pairs and take the groups of four coordinates of
// every staged step in turn (twice the waves for the same LDS traffic); their sums meet at the end.
template <bool CPLX>
__global__ __launch_bounds__(512) void k_pair_fwd(PairArgs a) {
    __shared__ __attribute__((aligned(16))) float Os[CPLX ? 2 : 1][PT][PPITCH];
    __shared__ __attribute__((aligned(16))) float Ns[CPLX ? 2 : 1][PT][PPITCH];
    __shared__ float halves[256][4];
    const int half = threadIdx.x >> 8, tid = threadIdx.x & 255;
    // pairs (ti + {0,16}, tj + {0,16}) of the tile: the 16 lanes with consecutive tj read consecutive staged rows,
    // which the row pitch spreads over all banks (rows 2 tj + {0,1} would fall on half of them)
    const int tj = tid & 15, ti = tid >> 4;
    const int j0 = blockIdx.x * PT, i0 = blockIdx.y * PT, c = blockIdx.z;
    const int NC = CPLX ? a.D / 2 : a.D;  // coordinates
    const float* Oc = a.O + (int64_t)c * a.g * a.D;
    const float* Nc = a.Nst + (int64_t)c * a.k * a.D;
    float acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
    const int lr = tid >> 3, lc = 4 * (tid & 7);
    // one thread stages one 16-byte piece per step (and per part): the first half of the workgroup the positives,
    // the second the negatives.  The piece for the next step is asked for before this step's arithmetic starts.
    const float* src = half == 0 ? Oc + (int64_t)(i0 + lr) * a.D : Nc + (int64_t)(j0 + lr) * a.D;
    const bool rok = half == 0 ? i0 + lr < a.g : j0 + lr < a.k;
    float (*dst)[PT][PPITCH] = half == 0 ? Os : Ns;
    float4 nxt[CPLX ? 2 : 1];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int part = 0; part < (CPLX ? 2 : 1); ++part) {
            nxt[part] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (rok && c0 + lc < NC) nxt[part] = ld4(src + part * NC + c0 + lc);  // NC is a multiple of 4
        }
    };
    fetch(0);
    for (int c0 = 0; c0 < NC; c0 += PCK) {
#pragma unroll
        for (int part = 0; part < (CPLX ? 2 : 1); ++part) st4(&dst[part][lr][lc], nxt[part]);
        if (c0 + PCK < NC) fetch(c0 + PCK);
        __syncthreads();
        // the 32 terms of this step are summed on their own and then added to the running total: the partial
        // sums stay small, which keeps the fp32 rounding of a 200- or 400-term sum near that of a pairwise sum
        float part[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
        for (int cq = 0; cq < PCK / 2; cq += 4) {
            // groups of four coordinates go to the two halves in turn, so that a last step with few coordinates is
            // still shared; (NC is a multiple of 4) what lies past NC is padding
            const int cc = 2 * cq + 4 * half;
            if (c0 + cc >= NC) break;
            float o_re[2][4], o_im[2][4], n_re[2][4], n_im[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float4 vo = ld4(&Os[0][ti + 16 * u][cc]), vn = ld4(&Ns[0][tj + 16 * u][cc]);
                o_re[u][0] = vo.x; o_re[u][1] = vo.y; o_re[u][2] = vo.z; o_re[u][3] = vo.w;
                n_re[u][0] = vn.x; n_re[u][1] = vn.y; n_re[u][2] = vn.z; n_re[u][3] = vn.w;
                if (CPLX) {
                    const float4 wo = ld4(&Os[CPLX ? 1 : 0][ti + 16 * u][cc]), wn = ld4(&Ns[CPLX ? 1 : 0][tj + 16 * u][cc]);
                    o_im[u][0] = wo.x; o_im[u][1] = wo.y; o_im[u][2] = wo.z; o_im[u][3] = wo.w;
                    n_im[u][0] = wn.x; n_im[u][1] = wn.y; n_im[u][2] = wn.z; n_im[u][3] = wn.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) { o_im[u][e] = 0.f; n_im[u][e] = 0.f; }
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) part[u][q] += pair_term<CPLX>(o_re[u][e], o_im[u][e], n_re[q][e], n_im[q][e]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) { acc[u][0] += part[u][0]; acc[u][1] += part[u][1]; }
        __syncthreads();
    }
    // padded coordinates hold zeros on both sides and contribute |0 - 0| = 0
    if (half == 1) {
        halves[tid][0] = acc[0][0]; halves[tid][1] = acc[0][1]; halves[tid][2] = acc[1][0]; halves[tid][3] = acc[1][1];
    }
    __syncthreads();
    if (half == 1) return;
    acc[0][0] += halves[tid][0]; acc[0][1] += halves[tid][1]; acc[1][0] += halves[tid][2]; acc[1][1] += halves[tid][3];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = i0 + ti + 16 * u, j = j0 + tj + 16 * q;
            if (i < a.g && j < a.k) a.S[((int64_t)c * a.g + i) * a.ld_s + j] = a.gamma - acc[u][q];
        }
    }
}

// ---- backward
// Workgroup: TI positives x a range of negatives x a range of `cpp` coordinates; thread (group, coordinate), the negatives
// are dealt round-robin to the `ng` groups.
struct PairBwdArgs {
    int n_i_tiles, i_parts;    // tiles of TI positives per chunk; workgroups that share them out (i_parts = n_i_tiles: one each)
    int n_j, tj;               // ranges of negatives per chunk, negatives per range
    int n_col, cpp;            // ranges of coordinates, coordinates per range
    int ng, tjb;               // thread groups; negatives per staged block of W (a multiple of ng)
    float* dstO;               // dL/do rows or their partial rows: [range of negatives][b x D]
    float* dstN;               // gradient rows of the corrupting entities or their partial rows: [i_parts][C*k x D]
    int64_t strideO, strideN;  // floats between consecutive partials (0: the final rows are written directly)
    // loss
    float alpha, invb;
    int ranking;
    const float* fpos;
    float* cpos;
    float* row_loss;
    float* loss_part;          // a sum per workgroup of the first range of coordinates
};

// What a wave needs to know of all scores of a positive: the maximum mx and the sum z of the softmax weights
// exp(alpha f - mx) / z (uniform weights: z = k), and, for the ranking loss, dL/df+ (only where `pos` is set).
template <bool LONG>
__device__ __forceinline__ void pair_row_stats(const PairBwdArgs& t, const float* s, int k, float gamma, bool pos, int64_t row, float& mx, float& z) {
    const int lane = threadIdx.x & 63;
    mx = 0.f;
    z = (float)k;
    if (!(t.alpha > 0.f) && !(t.ranking && pos)) return;  // (the same for every thread)
    if (t.alpha > 0.f) {
        mx = -INFINITY;
        for (int j0 = 0; j0 < k; j0 += 256) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = s[min(j0 + 64 * u + lane, k - 1)];
            mx = fmaxf(mx, t.alpha * fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
        }
        mx = wave_max(mx);
    }
    const float fp = t.fpos[row];
    z = 0.f;
    float on = 0.f;
    for (int j0 = 0; j0 < k; j0 += 256) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = s[min(j0 + 64 * u + lane, k - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (j0 + 64 * u + lane < k) {
                const float e = t.alpha > 0.f ? softmax_exp<LONG>(t.alpha * v[u] - mx) : 1.f;
                z += e;
                on += gamma - fp + v[u] > 0.f ? e : 0.f;
            }
        }
    }
    z = wave_sum(z);
    if (t.ranking && pos) {
        on = wave_sum(on);
        if (lane == 0) {
            t.cpos[row] = -(on / z) * t.invb;
            t.row_loss[row] = 0.f;  // (the gather launch left the logistic loss of the positive there)
        }
    }
}

// Bound by the vector ALUs (RotatE 13 issue slots per pair and coordinate, 4 of them the reciprocal square root; TransE-L1
// 4) plus about 8 us of launch, staging, the meeting of the groups' sums and the partial rows.  Measured per training
// step against workgroups that summed one side only, every term formed twice, behind a loss kernel (chunks of more than
// 128 positives took that form): RotatE g = b = 977, k = 92, D = 400 207 -> 53 us, TransE-L1 g = b = 579, k = 124, D = 176
// 163 -> 36 us, g = 601, k = 669, D = 408 293 -> 109 us; against tiles of 16 x 40 pairs of fixed shape: RotatE b = 1024, g = 128,
// k = 256, D = 400 78 -> 76 us, TransE-L1 b = 1440, g = 96, k = 138, D = 468 149 -> 80 us.
// Held to 128 registers: 16 wavefronts per CU, four on every SIMD.
// WALKS: a workgroup has several tiles of positives (where a set of partial rows for each would not fit the workspace).
// LONG: rows of more than KGE_SHORT_SCORES scores.
template <bool CPLX, int TI, bool WALKS, bool LONG>
__global__ __launch_bounds__(1024) void k_pair_bwd(PairArgs a, PairBwdArgs t) {
    constexpr int WPITCH = TI + 4;                 // floats per staged row of W^T
    constexpr int PART = CPLX ? 2 : 1;
    // TransE-L1: coordinates are held times 2^64, so that the clamp of a difference to [-w, w], w <= 1, is w sign(difference), 0
    // for 0: one v_med3 where two compares and two selects stood.  That holds if one of the two coordinates is 2^-40 or more
    // (they differ by 2^-64 then, or not at all); a thread compares where both may be smaller, and, unscaled, where one of
    // its o rows has a coordinate from 2^63 on.
    constexpr float SMALL = 0x1p24f;  // (2^-40, scaled)
    extern __shared__ __attribute__((aligned(16))) float lds[];  // W^T of the block [negative][WPITCH]; later group sums
    __shared__ float row_mx[TI], row_z[TI], row_li[16];
    const int tid = threadIdx.x, cpp = t.cpp, wave = tid >> 6, lane = tid & 63, n_waves = blockDim.x >> 6;
    const int grp = tid / cpp, lc = tid - grp * cpp;
    const int c = blockIdx.y;
    const int col = blockIdx.x % t.n_col, rest = blockIdx.x / t.n_col;
    const int ip = rest % t.i_parts, jt = rest / t.i_parts;
    const int jb0 = jt * t.tj, jb1 = min(jb0 + t.tj, a.k);
    const int NC = CPLX ? a.D / 2 : a.D;
    const int cc = col * cpp + lc;
    const bool act = grp < t.ng && cc < NC;
    const int ccs = act ? cc : 0;
    const float* Oc = a.O + (int64_t)c * a.g * a.D;
    const float* Nc = a.Nst + (int64_t)c * a.k * a.D;
    const float* Sc = a.S + (int64_t)c * a.g * a.ld_s;
    float* dN = t.dstN + ip * t.strideN + (int64_t)c * a.k * a.D;
    float* dO = t.dstO + jt * t.strideO + (int64_t)c * a.g * a.D + ccs;

    float li = 0.f;  // loss terms of the scores this thread turned into W
    for (int it = ip; it < t.n_i_tiles; it += WALKS ? t.i_parts : t.n_i_tiles) {
        const int i0 = it * TI, gi = min(TI, a.g - i0);
        float x_re[TI], x_im[CPLX ? TI : 1], g_re[TI], g_im[CPLX ? TI : 1];
#pragma unroll
        for (int s = 0; s < TI; ++s) {
            const float* po = Oc + (int64_t)(i0 + (s < gi ? s : 0)) * a.D + ccs;
            x_re[s] = po[0];
            g_re[s] = 0.f;
            if (CPLX) { x_im[s] = po[NC]; g_im[s] = 0.f; }
        }
        float scale = 1.f, y_least = 0.f;  // smallest |y| that all of x can be clamped against
        if (!CPLX) {
            bool large = false, small = false;
#pragma unroll
            for (int s = 0; s < TI; ++s) large |= !(fabsf(x_re[s]) < 0x1p63f);
            scale = large ? 1.f : 0x1p64f;
#pragma unroll
            for (int s = 0; s < TI; ++s) {
                x_re[s] *= scale;
                small |= fabsf(x_re[s]) < SMALL;
            }
            y_least = large ? INFINITY : small ? SMALL : 0.f;
        }
        for (int s = wave; s < gi; s += n_waves) {
            const int64_t row = (int64_t)c * a.g + i0 + s;
            float mx, z;
            pair_row_stats<LONG>(t, Sc + (int64_t)(i0 + s) * a.ld_s, a.k, a.gamma, jt == 0 && col == 0, row, mx, z);
            if (lane == 0) { row_mx[s] = mx; row_z[s] = z; }
        }
        for (int j0 = jb0; j0 < jb1; j0 += t.tjb) {
            const int jn = min(t.tjb, jb1 - j0);  // negatives in this block
            __syncthreads();
            // W = dL/df- of the block from the scores, transposed; a wave per positive; 0 for positives outside the chunk,
            // so that such pairs add nothing
            for (int s = wave; s < TI; s += n_waves) {
                const bool ok = s < gi;
                const float mx = ok ? row_mx[s] : 0.f, z = ok ? row_z[s] : 1.f;
                const float fp = ok && t.ranking ? t.fpos[(int64_t)c * a.g + i0 + s] : 0.f;
                const float* S = Sc + (int64_t)(i0 + (ok ? s : 0)) * a.ld_s + j0;
                for (int jb = lane; jb < jn; jb += 256) {
                    float f[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) f[u] = S[min(jb + 64 * u, jn - 1)];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        float w = (t.alpha > 0.f ? softmax_exp<LONG>(t.alpha * f[u] - mx) : 1.f) / z;
                        const bool on = ok && jb + 64 * u < jn;
                        if (t.ranking) {
                            const float m = a.gamma - fp + f[u];
                            li += on ? w * fmaxf(m, 0.f) : 0.f;
                            w = m > 0.f ? w * t.invb : 0.f;
                        } else {
                            float sp, sg;
                            softplus_sigmoid_of<LONG>(f[u], sp, sg);
                            li += on ? w * sp : 0.f;
                            w = w * sg * t.invb;
                        }
                        if (jb + 64 * u < jn) lds[(jb + 64 * u) * WPITCH + s] = ok ? w : 0.f;
                    }
                }
            }
            __syncthreads();
            if (grp >= jn || !act) continue;  // (the barriers above are outside of this)
            const char* nb = (const char*)(Nc + (int64_t)j0 * a.D);
            char* db = (char*)(dN + (int64_t)j0 * a.D);
            const uint32_t step = 4u * t.ng * a.D, last = 4u * ((jn - 1) * a.D + cc), im = 4u * NC;
            // rows are asked for two rounds before they are worked on: the store of the round before stands between a load
            // and its use, and waiting for that store would cost more than the round's arithmetic
            uint32_t off = 4u * (grp * a.D + cc);
            uint32_t nxt = min(off + step, last);
            float y_re = *(const float*)(nb + off) * scale, y_im = CPLX ? *(const float*)(nb + im + off) : 0.f;
            float y1_re = *(const float*)(nb + nxt), y1_im = CPLX ? *(const float*)(nb + im + nxt) : 0.f;
            for (int jj = grp; jj < jn; jj += t.ng) {
                float n_re = 0.f, n_im = 0.f;
                if (WALKS && it != ip) {  // on top of this workgroup's earlier tiles of positives
                    n_re = *(const float*)(db + off);
                    if (CPLX) n_im = *(const float*)(db + im + off);
                }
                nxt = min(nxt + step, last);
                const float z_re = *(const float*)(nb + nxt), z_im = CPLX ? *(const float*)(nb + im + nxt) : 0.f;
                if (!CPLX && !(fabsf(y_re) >= y_least)) {
#pragma unroll
                    for (int s = 0; s < TI; ++s) {
                        const float w = lds[jj * WPITCH + s], v = x_re[s] > y_re ? w : (x_re[s] < y_re ? -w : 0.f);
                        g_re[s] -= v;
                        n_re += v;
                    }
                } else {
#pragma unroll
                    for (int s4 = 0; s4 < TI; s4 += 4) {
                        const float4 w4 = ld4(&lds[jj * WPITCH + s4]);
                        const float wv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int s = s4 + e;
                            const float q_re = x_re[s] - y_re;  // o - n
                            if (CPLX) {
                                const float q_im = x_im[s] - y_im;
                                // w / |q|; q = 0 gives a finite factor times 0
                                const float f = wv[e] * __builtin_amdgcn_rsqf(fmaf(q_im, q_im, fmaf(q_re, q_re, 1.2e-38f)));
                                g_re[s] = fmaf(-f, q_re, g_re[s]);
                                g_im[s] = fmaf(-f, q_im, g_im[s]);
                                n_re = fmaf(f, q_re, n_re);
                                n_im = fmaf(f, q_im, n_im);
                            } else {
                                const float v = __builtin_amdgcn_fmed3f(q_re, -wv[e], wv[e]);
                                g_re[s] -= v;
                                n_re += v;
                            }
                        }
                    }
                }
                *(float*)(db + off) = n_re;
                if (CPLX) *(float*)(db + im + off) = n_im;
                off += step;
                y_re = y1_re * scale; y_im = y1_im;
                y1_re = z_re; y1_im = z_im;
            }
        }
        // dL/do: the groups' sums meet in LDS, the upper half of the groups added to the lower until one is left
        for (int left = t.ng; left > 1;) {
            const int half = (left + 1) / 2;
            __syncthreads();
            if (act && grp >= half && grp < left) {
                float* d = lds + (grp - half) * cpp + lc;
                const int pitch = (left - half) * cpp;
#pragma unroll
                for (int s = 0; s < TI; ++s) {
                    d[PART * s * pitch] = g_re[s];
                    if (CPLX) d[(PART * s + 1) * pitch] = g_im[s];
                }
            }
            __syncthreads();
            if (act && grp < left - half) {
                const float* d = lds + grp * cpp + lc;
                const int pitch = (left - half) * cpp;
#pragma unroll
                for (int s = 0; s < TI; ++s) {
                    g_re[s] += d[PART * s * pitch];
                    if (CPLX) g_im[s] += d[(PART * s + 1) * pitch];
                }
            }
            left = half;
        }
        if (grp == 0 && act) {
#pragma unroll
            for (int s = 0; s < TI; ++s) {
                if (s < gi) {
                    dO[(int64_t)(i0 + s) * a.D] = g_re[s];
                    if (CPLX) dO[(int64_t)(i0 + s) * a.D + NC] = g_im[s];
                }
            }
        }
        __syncthreads();  // (the next tile of positives stages its W where the sums were)
    }
    if (col != 0) return;
    li = wave_sum(li);
    if (lane == 0) row_li[wave] = li;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < n_waves; ++w) li += row_li[w];
        t.loss_part[((int64_t)c * t.n_j + jt) * t.i_parts + ip] = li * t.invb;
    }
}

}  // namespace

void kge_pair_neg_score(kge_ctx* c, int b, int k, int gsz, float gamma, float* out, int ld_out, hipStream_t st) {
    PairArgs a = {};
    a.O = c->O; a.Nst = c->Nst; a.S = out; a.ld_s = ld_out; a.g = gsz; a.k = k; a.D = c->cfg.ent_dim; a.gamma = gamma;
    const dim3 grid((k + PT - 1) / PT, (gsz + PT - 1) / PT, b / gsz);
    if (c->cfg.model == KGE_ROTATE) KGE_LAUNCH(c, k_pair_fwd<true>, grid, dim3(512), 0, st, a);
    else KGE_LAUNCH(c, k_pair_fwd<false>, grid, dim3(512), 0, st, a);
}

int kge_pair_neg_backward(kge_ctx* c, int b, int k, int gsz, float gamma, hipStream_t st) {
    PairArgs a = {};
    a.O = c->O; a.Nst = c->Nst; a.S = c->S; a.ld_s = c->ld_s; a.g = gsz; a.k = k; a.D = c->cfg.ent_dim; a.gamma = gamma;
    const int chunks = b / gsz;
    PairBwdPlan& p = c->pair_plan;
    if (p.b != b || p.k != k || p.g != gsz) p = plan_pair_bwd(c->cfg.model == KGE_ROTATE, a.D, c->pair_part_n_floats, b, k, gsz);
    float* Gneg = c->Gent + (int64_t)2 * b * a.D;
    const int64_t rows_o = (int64_t)b * a.D, rows_n = (int64_t)chunks * k * a.D;
    PairBwdArgs t;
    t.n_i_tiles = p.n_i; t.i_parts = p.i_parts; t.n_j = p.pj; t.tj = p.tj; t.n_col = p.n_col; t.cpp = p.cpp; t.ng = p.ng;
    t.tjb = pair_bwd_block(p.ti, p.ng, p.tj);
    t.dstO = p.pj > 1 ? c->pair_part_o : c->GO;
    t.strideO = p.pj > 1 ? rows_o : 0;
    t.dstN = p.i_parts > 1 ? c->pair_part_n : Gneg;
    t.strideN = p.i_parts > 1 ? rows_n : 0;
    t.alpha = c->cfg.adv_temperature; t.invb = 1.f / (float)b; t.ranking = c->cfg.loss == KGE_LOSS_RANKING;
    t.fpos = c->fpos; t.cpos = c->cpos; t.row_loss = c->row_loss; t.loss_part = c->neg_loss_part;
    const bool cplx = c->cfg.model == KGE_ROTATE;
    const int lds = pair_bwd_lds(cplx, p.ti, p.ng, p.cpp, t.tjb);
    const dim3 grid(p.i_parts * p.pj * p.n_col, chunks), block((p.ng * p.cpp + 63) / 64 * 64);
    const bool walks = p.i_parts < p.n_i;
#define KGE_BWD(CPLX, TI, WALKS)                                                                              \
    do {                                                                                                      \
        if (k > KGE_SHORT_SCORES) KGE_LAUNCH(c, (k_pair_bwd<CPLX, TI, WALKS, true>), grid, block, lds, st, a, t); \
        else KGE_LAUNCH(c, (k_pair_bwd<CPLX, TI, WALKS, false>), grid, block, lds, st, a, t);                 \
    } while (0)
    if (cplx) {
        if (walks) KGE_BWD(true, 16, true);
        else if (p.ti == 8) KGE_BWD(true, 8, false);
        else KGE_BWD(true, 16, false);
    } else {
        if (walks) KGE_BWD(false, 16, true);
        else if (p.ti == 8) KGE_BWD(false, 8, false);
        else if (p.ti == 16) KGE_BWD(false, 16, false);
        else KGE_BWD(false, 32, false);
    }
#undef KGE_BWD
    // the chain launch that follows adds up the partial rows
    c->go_partial = {c->pair_part_o, c->GO, p.pj, rows_o, rows_o / 4};
    c->neg_partial = {c->pair_part_n, Gneg, p.i_parts, rows_n, rows_n / 4};
    return p.i_parts * p.pj * chunks;
}
