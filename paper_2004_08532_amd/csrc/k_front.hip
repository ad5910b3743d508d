// Gather and forward product in one launch, for steps of few output tiles.
//
// The forward product needs o_i = phi(a_i, r_i) and the corrupting rows; the gather launch forms and stages them, and a
// second launch reads them back.  Where the output has few tiles (the chip holds 512 of these workgroups, two per CU by their LDS;
// the limits, 384 to 768 tiles, are measured: kge_front_fits) the tiles can read the table rows themselves: a workgroup of eight waves owns a 32 x 32 output tile, every wave asks for whole rows (of four
// positives and four corrupting entities) in one round, forms o, and lays both operands out in LDS in slices of 256 floats
// of K, which the waves then split between them.  The tiles stage the corrupting rows for the backward
// product; o rows, the scores of the positives and the key order come from other workgroups of the launch
// (k_gather_rows.h), which need nothing from the tiles.  What it saves is the ramp and the drain of a launch and a round
// trip through memory: gather + forward 8.0 + 7.2 -> 13.4 us at Freebase scale, 8.3 + 6.7 -> 11.1 FB15k-sized (D 400),
// 5.1 + 5.3 -> 6.9 in a step of 256 positives (D 64).
// TransE-L1 forms its sums of absolute differences from the same staged rows.  (RotatE has not been tried here: every tile would
// form the sines and cosines of its 32 relation rows again.)
#include "k_gather_rows.h"
#include "k_gemm_shared.h"

namespace {

constexpr int FT = 512, FW = FT / 64, TILE = 32;
constexpr int RPW = TILE / FW;   // rows of either operand per wave
constexpr int SLICE = 256;       // floats of K in LDS at a time
constexpr int PITCH = SLICE + 4;  // floats; 16-byte reads of 16 consecutive rows fall into different banks
constexpr int FRONT_MAX_KEYS = 8192;  // (they lie in the LDS of the tiles)
static_assert(FRONT_MAX_KEYS <= 2 * TILE * PITCH && FW * TILE * TILE + FW * 2 * TILE + FW <= 2 * TILE * PITCH, "LDS");

struct FrontArgs {
    GatherArgs ga;
    float* C;
    int ldc, g, k;
    int gx, gy, tiles, per_xcd;
    int rank_wgs;  // rank blocks, rounded up to a multiple of 8
    int out_mode;  // TransE-L1: OUT_SCORE; others (training steps only): OUT_DIST or OUT_W
    bool stage;    // training: stage the corrupting rows
    float wk;
    float* neg_loss_part;
};

// sum of the eight waves' values `stride` floats apart, in pairs
__device__ __forceinline__ float sum_of_waves(const float* p, int stride) {
    float v[FW];
#pragma unroll
    for (int w = 0; w < FW; ++w) v[w] = p[w * stride];
    return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

// One 32 x 32 tile.  Bound by the round trips kernel arguments -> ids -> rows (2.1 us of a tile's 9 at Freebase scale: 224 tiles,
// D 400) and by the matrix cores (1.5 us: a CU holds one tile, whose products take 3,200 cycles on its four SIMDs).  Every wave
// reads whole rows, all of them in flight together: tiles that read their K ranges of the rows piece by piece took twice as
// long.  Two slices of K, so that two workgroups share a CU's LDS and the second slice arrives while the first is multiplied.
template <int MODEL, int NV>
__device__ __forceinline__ void front_tile(const FrontArgs& f, int tile, float* lds) {
    constexpr bool CPLX = MODEL == KGE_COMPLEX;
    constexpr int P = CPLX ? 2 * NV : NV;  // slices of K (ComplEx: real and imaginary parts of 256 coordinates)
    static_assert(!CPLX || NV == 1, "the two halves of a row are a slice each");
    const GatherArgs& a = f.ga;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, D = a.D;
    const int n0 = (tile % f.gx) * TILE, m0 = (tile / f.gx) % f.gy * TILE, c = tile / (f.gx * f.gy);
    const StepView sv = step_view(a.ids);
    const bool head = sv.side == KGE_NEG_HEAD;
    float* As = lds;
    float* Bs = lds + TILE * PITCH;
    const int half = D / 2;
    auto width = [&](int p) { return CPLX ? half : min(SLICE, D - SLICE * p); };
    auto piece = [&](int p) { return (CPLX ? half : SLICE) * p + (4 * lane < width(p) ? 4 * lane : 0); };

    // rows past the end of the matrix: the last row again, dropped in the epilogue
    float4 A[RPW][P], R[RPW][P], N[RPW][P];
    const float *pa[RPW], *pr[RPW], *pn[RPW];
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
        const int i = c * f.g + min(m0 + w + FW * q, f.g - 1), j = c * f.k + min(n0 + w + FW * q, f.k - 1);
        pn[q] = a.E + clamp_id(sv.neg[j], a.n_ent) * (int64_t)D;
        if (MODEL == KGE_RESCAL) {
            pa[q] = a.O + (int64_t)i * D;
        } else {
            pa[q] = a.E + clamp_id(head ? sv.t[i] : sv.h[i], a.n_ent) * (int64_t)D;
            pr[q] = a.R + clamp_id(sv.r[i], a.n_rel) * (int64_t)a.Dr;
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            A[q][p] = ld4(pa[q] + piece(p));
            if (MODEL != KGE_RESCAL) R[q][p] = ld4(pr[q] + piece(p));
            N[q][p] = ld4(pn[q] + piece(p));
        }
    }
    if constexpr (CPLX) {
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const float4 x = A[q][0], y = A[q][1], u = R[q][0];
            float4 v = R[q][1];
            if (head) v = make_float4(-v.x, -v.y, -v.z, -v.w);  // o = t conj(r)
            A[q][0] = make_float4(x.x * u.x - y.x * v.x, x.y * u.y - y.y * v.y, x.z * u.z - y.z * v.z, x.w * u.w - y.w * v.w);
            A[q][1] = make_float4(x.x * v.x + y.x * u.x, x.y * v.y + y.y * u.y, x.z * v.z + y.z * u.z, x.w * v.w + y.w * u.w);
        }
    }
    // the corrupting rows for the backward product: the (up to four) rows of tiles share the work of staging them
    const int by = m0 / TILE, sharers = min(f.gy, RPW);
    auto stages = [&](int q) { return f.stage && q % sharers == by && n0 + w + FW * q < f.k; };
    floatx16 acc = {}, acc2 = {};  // (two, so that a sum is a chain of half the length)
    float sums[2][2] = {{0.f, 0.f}, {0.f, 0.f}};  // TransE-L1
    float on = 0.f, nn = 0.f;  // TransE-L2: |o|^2 and |n|^2 of row lane % 32 over this lane's part of K
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const bool in = 4 * lane < width(p);
        if (p > 0) __syncthreads();
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            float4 o = A[q][p], n = N[q][p];
            const float4 r = R[q][p];
            if (MODEL == KGE_DISTMULT) o = make_float4(o.x * r.x, o.y * r.y, o.z * r.z, o.w * r.w);
            if (MODEL == KGE_TRANSE_L2 || MODEL == KGE_TRANSE_L1) {
                o = head ? make_float4(o.x - r.x, o.y - r.y, o.z - r.z, o.w - r.w)
                         : make_float4(o.x + r.x, o.y + r.y, o.z + r.z, o.w + r.w);
            }
            o = in ? o : f4(0.f);
            if (stages(q) && in) st4(a.Nst + (int64_t)(c * f.k + n0 + w + FW * q) * D + piece(p), n);
            n = in ? n : f4(0.f);
            st4(As + (w + FW * q) * PITCH + 4 * lane, o);
            st4(Bs + (w + FW * q) * PITCH + 4 * lane, n);
        }
        __syncthreads();
        if constexpr (MODEL == KGE_TRANSE_L1) {
            // pairs (ti + {0,16}, tj + {0,16}); the two halves of the workgroup take groups of four coordinates in turn.  32
            // coordinates are summed on their own, then added to the total: the order of k_pair_fwd, bit for bit
            for (int c0 = 0; c0 < width(p); c0 += 32) {
                float part[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
                for (int cq = 0; cq < 32; cq += 8) {
                    const int cc = c0 + cq + 4 * (threadIdx.x >> 8);
                    if (cc >= width(p)) break;
                    float4 o[2], n[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        o[u] = ld4(As + ((threadIdx.x >> 4 & 15) + 16 * u) * PITCH + cc);
                        n[u] = ld4(Bs + ((threadIdx.x & 15) + 16 * u) * PITCH + cc);
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            part[u][q] += fabsf(o[u].x - n[q].x);
                            part[u][q] += fabsf(o[u].y - n[q].y);
                            part[u][q] += fabsf(o[u].z - n[q].z);
                            part[u][q] += fabsf(o[u].w - n[q].w);
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) { sums[u][0] += part[u][0]; sums[u][1] += part[u][1]; }
            }
            continue;
        }
        const int octets = (width(p) + 7) / 8;
        const float* ra = As + (lane & 31) * PITCH + 4 * (lane >> 5);
        const float* rb = Bs + (lane & 31) * PITCH + 4 * (lane >> 5);
        for (int q = w; q < octets; q += FW) {
            const float4 x = ld4(ra + 8 * q), y = ld4(rb + 8 * q);
            if (MODEL == KGE_TRANSE_L2) {
                on += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
                nn += y.x * y.x + y.y * y.y + y.z * y.z + y.w * y.w;
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, acc, 0, 0, 0);
            acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, acc2, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, acc, 0, 0, 0);
            acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, acc2, 0, 0, 0);
        }
    }
    __syncthreads();
    if constexpr (MODEL == KGE_TRANSE_L1) {
        float* C = f.C + (int64_t)c * f.g * f.ldc;
        float* other = lds + 4 * (threadIdx.x & 255);
        if (threadIdx.x >= 256) st4(other, make_float4(sums[0][0], sums[0][1], sums[1][0], sums[1][1]));
        __syncthreads();
        if (threadIdx.x >= 256) return;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int i = m0 + (threadIdx.x >> 4) + 16 * u, j = n0 + (threadIdx.x & 15) + 16 * q;
                if (i < f.g && j < f.k) C[(int64_t)i * f.ldc + j] = a.gamma - (sums[u][q] + other[2 * u + q]);
            }
        }
        return;
    }
    // sums of the waves (in wave order) and the norms
    float* norms = lds + FW * TILE * TILE;
    if (MODEL == KGE_TRANSE_L2) {
        on += __shfl_xor(on, 32, 64);
        nn += __shfl_xor(nn, 32, 64);
        norms[w * 2 * TILE + lane] = lane < 32 ? on : nn;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) lds[w * TILE * TILE + (8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * TILE + (lane & 31)] = acc[v] + acc2[v];
    __syncthreads();
    float loss = 0.f;
    float* C = f.C + (int64_t)c * f.g * f.ldc;
#pragma unroll
    for (int it = 0; it < TILE * TILE / FT; ++it) {
        const int e = threadIdx.x + it * FT, gm = m0 + (e >> 5), gn = n0 + (e & 31);
        if (gm >= f.g || gn >= f.k) continue;
        const float s = sum_of_waves(lds + e, TILE * TILE);
        float out;
        if (MODEL == KGE_TRANSE_L2) {
            const float o2 = sum_of_waves(norms + (e >> 5), 2 * TILE), n2 = sum_of_waves(norms + TILE + (e & 31), 2 * TILE);
            const float d = sqrtf(fmaxf(o2 + n2 - 2.f * s, 0.f));
            out = d;
            if (f.out_mode == OUT_W) {
                const float coef = w_and_loss<true>(a.gamma - d, f.wk, loss);
                out = d > 0.f ? coef * __builtin_amdgcn_rcpf(d) : 0.f;
            }
        } else {
            out = f.out_mode == OUT_W ? w_and_loss<true>(s, f.wk, loss) : s;
        }
        C[(int64_t)gm * f.ldc + gn] = out;
    }
    if (f.out_mode == OUT_W) {
        loss = wave_sum(loss);
        float* part = norms + FW * 2 * TILE;
        if (lane == 0) part[w] = loss;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
#pragma unroll
            for (int ww = 0; ww < FW; ++ww) t += part[ww];
            f.neg_loss_part[tile] = t * f.wk;
        }
    }
}

template <int MODEL, int NV>
__global__ __launch_bounds__(FT) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_front(FrontArgs f) {
    __shared__ __attribute__((aligned(16))) uint32_t front_lds[2 * TILE * PITCH];
    int block = blockIdx.x;
    if (block < f.rank_wgs) {
        const GatherArgs& a = f.ga;
        if (block < a.ent_rank_blocks) rank_block<FT>(a.ent, block, front_lds);
        else if (block < a.rank_blocks) rank_block<FT>(a.rel, block - a.ent_rank_blocks, front_lds);
        return;
    }
    block -= f.rank_wgs;
    if (block < 8 * f.per_xcd) {
        const int tile = xcd_tile(block >> 3, f.per_xcd);
        if (tile < f.tiles) front_tile<MODEL, NV>(f, tile, reinterpret_cast<float*>(front_lds));
        return;
    }
    const int row = (block - 8 * f.per_xcd) * FW + (threadIdx.x >> 6);
    if (row < f.ga.b) gather_row<MODEL, NV>(f.ga, row);  // (positives, fp32: the tiles stage the corrupting rows)
}

}  // namespace

// Forward of chunks of gsz positives and k corrupting rows in the gather launch?
// Tiles read a table row once per tile that needs it, the gather launch once, so the line lies where that costs more than a
// launch (us per training step, separate -> one launch; chunks of 128 where nothing else is said):
//   TransE-L2   rows of 400: 256 tiles 41.7 -> 37.9, 640 66.0 -> 61.0, 1024 66.9 -> 67.1;  of 160: 512 43.0 -> 41.3, 576 46.8 ->
//               44.5;  of 128: 624 40.3 -> 39.1, 640 43.4 -> 43.6, 768 44.6 -> 46.7
//   DistMult    rows of 400: 640 64.0 -> 62.8, 768 67.9 -> 67.5;  of 160: 768 51.2 -> 48.6;  of 128: 512 39.4 -> 36.4, 624 42.3 ->
//               40.9;  of 64: 512 37.1 -> 33.6
//   RESCAL      rows of 200: 256 87.9 -> 83.6, 768 (chunks of 256) 103.3 -> 97.9;  of 64: 512 57.2 -> 52.4
//   TransE-L1   rows of 400: 256 61.4 -> 57.2, 704 103.6 -> 99.3;  of 160: 576 62.4 -> 60.5, 704 67.7 -> 70.2;  of 64: 416 47.6 ->
//               46.3, 512 48.6 -> 46.3
//   ComplEx     rows of 400: 256 39.9 -> 36.3, 576 62.2 -> 58.0, 768 (chunks of 256) 62.3 -> 57.4;  of 256: 384 42.1 -> 40.9, 512
//               45.0 -> 46.9;  of 160: 384 37.7 -> 37.0, 512 41.6 -> 43.5, 640 47.1 -> 51.3;  of 64: 384 33.0 -> 32.4, 512 37.3 ->
//               38.7 (its halves are a slice each, and these are at most half full there)
//   keys        ordered by brute force here, in buckets of the id range in the gather launch of long lists (512 tiles and
//               fewer, rows of 64): 6144 39.1 -> 35.4, 8192 40.6 -> 34.7, 12288 45.0 -> 47.9.  With more tiles than that they add to a
//               launch that is several rounds long: TransE-L2 rows of 400 7168 keys 66.0 -> 61.0, 7680 68.4 -> 70.0, 8192 70.2 -> 72.1,
//               rows of 160 7168 48.9 -> 49.1, 8192 51.3 -> 53.5, ComplEx rows of 400 6912 63.0 -> 61.5, 7168 63.8 -> 65.2, 7680
//               66.4 -> 68.0;  not so with the others, whose tiles need fewer registers (DistMult 7680 66.3 -> 65.7, rows of 200 8192
//               53.0 -> 49.8; TransE-L1 and RESCAL above).  Lists that are sorted in other launches don't matter: 20480 keys
//               67.8 -> 67.3
// Rows of more than two slices of K would not fit the registers of a wave.
bool kge_front_fits(const kge_ctx* c, int b, int k, int gsz, bool with_keys) {
    const int m = c->cfg.model, D = c->cfg.ent_dim;
    if (c->cfg.gemm_input != 0 || D > 2 * SLICE) return false;
    if (m != KGE_TRANSE_L2 && m != KGE_TRANSE_L1 && m != KGE_DISTMULT && m != KGE_COMPLEX && m != KGE_RESCAL) return false;
    const int64_t chunks = b / gsz, tiles = chunks * ((gsz + TILE - 1) / TILE) * ((k + TILE - 1) / TILE);
    const int64_t most_tiles = m == KGE_COMPLEX && D <= SLICE ? 384 : D > 128 ? 768 : 512;
    const int64_t most_keys = (m == KGE_TRANSE_L2 || m == KGE_COMPLEX) && tiles > 512 ? 7168 : FRONT_MAX_KEYS;
    return tiles <= most_tiles && !(with_keys && 2 * (int64_t)b + chunks * k > most_keys);
}

void kge_launch_front(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, int gsz, float gamma, float* pos_out,
                      bool train, bool with_keys, float* out, int ld_out, int out_mode, hipStream_t st) {
    FrontArgs f = {};
    kge_fill_gather_args(c, E, R, ids, gsz, gamma, pos_out, &f.ga);
    f.C = out; f.ldc = ld_out; f.g = gsz; f.k = k;
    f.gx = (k + TILE - 1) / TILE; f.gy = (gsz + TILE - 1) / TILE; f.tiles = f.gx * f.gy * (ids.b / gsz);
    f.per_xcd = (f.tiles + 7) / 8;
    f.out_mode = out_mode;
    f.wk = 1.f / ((float)k * (float)ids.b);
    f.neg_loss_part = c->neg_loss_part;
    f.stage = train;
    if (with_keys) {
        constexpr int ITEMS = RankShape<FT>::ITEMS;
        kge_make_key_lists(c, ids, &f.ga.ent, &f.ga.rel);
        f.ga.ent_rank_blocks = (f.ga.ent.n + ITEMS - 1) / ITEMS;
        f.ga.rank_blocks = f.ga.ent_rank_blocks + (f.ga.rel.n + ITEMS - 1) / ITEMS;
        f.rank_wgs = (f.ga.rank_blocks + 7) / 8 * 8;
        c->ebuf = 0;
        c->rbuf = 0;
    }
    const dim3 grid(f.rank_wgs + 8 * f.per_xcd + (ids.b + FW - 1) / FW);
    const int nv = (c->cfg.ent_dim + SLICE - 1) / SLICE;
    switch (c->cfg.model) {
    case KGE_TRANSE_L2:
        if (nv == 1) KGE_LAUNCH(c, (k_front<KGE_TRANSE_L2, 1>), grid, dim3(FT), 0, st, f);
        else KGE_LAUNCH(c, (k_front<KGE_TRANSE_L2, 2>), grid, dim3(FT), 0, st, f);
        break;
    case KGE_TRANSE_L1:
        if (nv == 1) KGE_LAUNCH(c, (k_front<KGE_TRANSE_L1, 1>), grid, dim3(FT), 0, st, f);
        else KGE_LAUNCH(c, (k_front<KGE_TRANSE_L1, 2>), grid, dim3(FT), 0, st, f);
        break;
    case KGE_DISTMULT:
        if (nv == 1) KGE_LAUNCH(c, (k_front<KGE_DISTMULT, 1>), grid, dim3(FT), 0, st, f);
        else KGE_LAUNCH(c, (k_front<KGE_DISTMULT, 2>), grid, dim3(FT), 0, st, f);
        break;
    case KGE_RESCAL:
        if (nv == 1) KGE_LAUNCH(c, (k_front<KGE_RESCAL, 1>), grid, dim3(FT), 0, st, f);
        else KGE_LAUNCH(c, (k_front<KGE_RESCAL, 2>), grid, dim3(FT), 0, st, f);
        break;
    default: KGE_LAUNCH(c, (k_front<KGE_COMPLEX, 1>), grid, dim3(FT), 0, st, f); break;
    }
}
