// The fp32 product S_c = O_c N_c^T of k_gemm.hip on larger tiles, bit for bit.
//
// k_gemm_fwd gives every 32 x 32 tile to a workgroup of its own, whose waves take every fourth block of K: a tile pulls 64 rows through
// the L1s for 32 x 32 scores, 2 KB per 64 matrix cycles of a CU, and that path, not the matrix cores, sets its pace.  Here four waves
// share the rows of a 64 x 64 tile through LDS (half the bytes), and a wave owns a 32 x 32 block of it over the whole of K.  A rank
// hangs on the last bit of a score (split_forward in k_gemm.hip), so the sums keep their order: block kb of K goes into
// accumulator kb mod 4, as it would into that wave of k_gemm_fwd, and the four are added up in order.
// What bounds it: matrix instructions.  1000 x 2000 x 400 (two workgroups per CU): 46.4 -> 30.4 us for kge_rank with its metrics, the
// product 36 -> 22 by itself, of which the matrix instructions take 13 at the 2.07 GHz that the clock shows in it (2048 of about
// 2550 cycles per block of K); 4000 cycles pass before the first block is there, 3600 behind the last.  Ranks: one global atomic per row
// and tile instead of one per row and 32 columns (D 64: 35.9 -> 16.9 us).  Tiles of 64 x 128 (a CU each at this size) take 1 us more, of 128 x
// 128 11.5 (half of the CUs), of 32 x 128 1.5; operands read from LDS before they are multiplied, without the second set: 2.6.
#include "k_gemm_shared.h"

namespace {

constexpr int NW = 4;  // waves of k_gemm_fwd whose sums these are
constexpr int BK = 32, PITCH = 36;  // K block; floats per LDS row: 16-byte aligned, 128-bit reads of eight rows free of conflicts

constexpr int BM = 64, BN = 64;              // output tile
constexpr int THREADS = BM / 32 * (BN / 32) * 64;
constexpr int STEP = THREADS / 8;            // rows that the threads load together, 16 bytes each
constexpr int RA = BM / STEP, RB = BN / STEP;
constexpr int P = 2;                         // blocks of K in flight (four: no change)

__device__ __forceinline__ void lds_barrier() {  // orders LDS traffic only: global loads stay in flight across it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int EPI>
__global__ __launch_bounds__(THREADS) void k_gemm_fwd_wide(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) float lds[2][(BM + BN) * PITCH];
    __shared__ float row_norm[BM], row_score[BM];
    __shared__ int row_count[BM];
    const int tile = xcd_tile(blockIdx.x >> 3, gridDim.x >> 3);
    if (tile >= g.tiles) return;
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const int n0 = (tile % g.gx) * BN, m0 = (tile / g.gx) % g.gy * BM, c = tile / (g.gx * g.gy);
    const int wm = 32 * (w / (BN / 32)), wn = 32 * (w % (BN / 32));  // this wave's block of the tile

    // rows past the end of the matrix: the last row again, dropped in the epilogue.  K values past the end become zeros.
    const int row = t >> 3, piece = t & 7;
    const float *pa[RA], *pb[RB];
#pragma unroll
    for (int q = 0; q < RA; ++q) pa[q] = g.A + c * g.sA + (int64_t)min(m0 + row + STEP * q, g.M - 1) * g.lda;
#pragma unroll
    for (int q = 0; q < RB; ++q) pb[q] = g.B + c * g.sB + (int64_t)min(n0 + row + STEP * q, g.N - 1) * g.ldb;
    struct Block { float4 a[RA], b[RB]; };
    auto issue = [&](int kb) {
        const int k = kb * BK + 4 * piece, at = k < g.K ? k : 0;
        Block r;
#pragma unroll
        for (int q = 0; q < RA; ++q) r.a[q] = ld4(pa[q] + at);
#pragma unroll
        for (int q = 0; q < RB; ++q) r.b[q] = ld4(pb[q] + at);
        return r;
    };
    auto store = [&](int kb, const Block& r, float* buf) {
        const bool in = kb * BK + 4 * piece < g.K;  // (K is a multiple of 4)
#pragma unroll
        for (int q = 0; q < RA; ++q) st4(buf + (row + STEP * q) * PITCH + 4 * piece, in ? r.a[q] : f4(0.f));
#pragma unroll
        for (int q = 0; q < RB; ++q) st4(buf + (BM + row + STEP * q) * PITCH + 4 * piece, in ? r.b[q] : f4(0.f));
    };
    floatx16 acc[NW] = {};
    // A lane's K values of a block: kk = 8 q + 4 (lane / 32) + e, q, e = 0 .. 3
    struct Operands { float4 a[BK / 8], b[BK / 8]; };
    const int at_a = (wm + (lane & 31)) * PITCH + 4 * (lane >> 5), at_b = (BM + wn + (lane & 31)) * PITCH + 4 * (lane >> 5);
    auto mfma = [&](const float4& a, const float4& b, int e, floatx16& acc) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(e == 0 ? a.x : e == 1 ? a.y : e == 2 ? a.z : a.w,
                                                   e == 0 ? b.x : e == 1 ? b.y : e == 2 ? b.z : b.w, acc, 0, 0, 0);
    };
    const int nblk = (g.K + BK - 1) / BK;
    Block r[P];
#pragma unroll
    for (int p = 0; p < P; ++p) r[p] = issue(p);
    // what the epilogue wants of the rows
    const int my_row = min(m0 + t % BM, g.M - 1);
    const float my_norm = EPI == EPI_L2_FWD ? g.rowv[c * g.s_rowv + my_row] : 0.f;
    const float my_score = g.out_mode == OUT_RANK ? g.fpos[c * g.M + my_row] : 0.f;
    const int gn = n0 + wn + (lane & 31);
    const float col_norm = EPI == EPI_L2_FWD ? g.colv[c * g.s_colv + min(gn, g.N - 1)] : 0.f;
    Operands f[2];
    store(0, r[0], lds[0]);
    r[0] = issue(P);
    lds_barrier();
#pragma unroll
    for (int q = 0; q < BK / 8; ++q) { f[0].a[q] = ld4(lds[0] + at_a + 8 * q); f[0].b[q] = ld4(lds[0] + at_b + 8 * q); }
    // Block base + p is multiplied from registers.  Meanwhile the next one goes to LDS, and from there, a read behind every matrix
    // instruction, into the other set of operands (past the last one zeros go that way).
    auto step = [&](int base, int p) {
        store(base + p + 1, r[(p + 1) % P], lds[(p + 1) & 1]);
        r[(p + 1) % P] = issue(base + p + 1 + P);
        const Operands& now = f[p & 1];
        Operands& next = f[(p + 1) & 1];
#pragma unroll
        for (int i = 0; i < 8; ++i) mfma(now.a[i >> 2], now.b[i >> 2], i & 3, acc[p]);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mfma(now.a[2 + (i >> 2)], now.b[2 + (i >> 2)], i & 3, acc[p]);
            if (i & 1) next.b[i >> 1] = ld4(lds[(p + 1) & 1] + at_b + 8 * (i >> 1));
            else next.a[i >> 1] = ld4(lds[(p + 1) & 1] + at_a + 8 * (i >> 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int base = 0;
    for (; base + NW <= nblk; base += NW) {
#pragma unroll
        for (int p = 0; p < NW; ++p) step(base, p);
    }
#pragma unroll
    for (int p = 0; p < NW - 1; ++p) {
        if (base + p >= nblk) break;
        step(base, p);
    }
    if (t < BM) {
        row_norm[t] = my_norm;
        row_score[t] = my_score;
        row_count[t] = 0;
    }
    __syncthreads();

    // ---- epilogue: register v of lane l holds element (8 (v/4) + 4 (l/32) + v%4, l%32) of the wave's block
    auto row_of = [&](int v) { return wm + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); };
    float* C = g.C + c * g.sC;
    float loss = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int lr = row_of(v), gm = m0 + lr;
        const bool in = gm < g.M && gn < g.N;
        float s = 0.f + acc[0][v], d = 0.f;
#pragma unroll
        for (int p = 1; p < NW; ++p) s += acc[p][v];
        if (EPI == EPI_L2_FWD) {
            const float d2 = row_norm[lr] + col_norm - 2.f * s;
            d = sqrtf(fmaxf(d2, 0.f));
            s = g.gamma - d;
        }
        if (g.out_mode == OUT_RANK) {  // rank_i = 1 + #{j : f-_ij > f+_i}: a half wave counts its columns
            const unsigned long long m = __ballot(in && s > row_score[lr]);
            const int cnt = __popcll(lane < 32 ? m & 0xffffffffull : m >> 32);
            if ((lane & 31) == 0 && cnt > 0) atomicAdd(&row_count[lr], cnt);
            continue;
        }
        if (!in) continue;
        if (g.out_mode == OUT_W) {  // W = w sigmoid(f) [/ |o - n|, 0 where the distance is 0]
            s = w_and_loss<true>(s, g.wk, loss);
            if (EPI == EPI_L2_FWD) s = d > 0.f ? s * __builtin_amdgcn_rcpf(d) : 0.f;
        } else if (EPI == EPI_L2_FWD && g.out_mode == OUT_DIST) {
            s = d;
        }
        C[(int64_t)gm * g.ldc + gn] = s;
    }
    if (g.out_mode == OUT_W) {
        // negative part of the loss, one sum per 32 x 32 block that lies inside the matrix, indexed as 32 x 32 tiles are
        loss = wave_sum(loss);
        const int bm = (m0 + wm) / 32, bn = (n0 + wn) / 32, nx = (g.N + 31) / 32, ny = (g.M + 31) / 32;
        if (lane == 0 && bm < ny && bn < nx) g.neg_loss_part[(c * ny + bm) * nx + bn] = loss * g.wk;
    } else if (g.out_mode == OUT_RANK) {  // one integer atomic per row and tile, any order
        __syncthreads();
        if (t < BM && m0 + t < g.M && row_count[t] > 0) atomicAdd(&g.rank[c * g.M + m0 + t], row_count[t]);
    }
}

template <int EPI>
void launch(kge_ctx* c, GemmArgs g, int chunks, hipStream_t st) {
    g.gx = (g.N + BN - 1) / BN;
    g.gy = (g.M + BM - 1) / BM;
    g.tiles = g.gx * g.gy * chunks;
    KGE_LAUNCH(c, k_gemm_fwd_wide<EPI>, dim3(8 * ((g.tiles + 7) / 8)), dim3(THREADS), 0, st, g);
}

}  // namespace

void kge_gemm_wide_forward(kge_ctx* c, const void* args, int epi, int chunks, hipStream_t st) {
    const GemmArgs& g = *static_cast<const GemmArgs*>(args);
    if (epi == EPI_L2_FWD) launch<EPI_L2_FWD>(c, g, chunks, st);
    else launch<EPI_PLAIN>(c, g, chunks, st);
}
