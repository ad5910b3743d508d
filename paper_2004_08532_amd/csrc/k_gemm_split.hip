// The forward product S_c = O_c N_c^T of training steps with many output tiles: fp32 operands on the bf16 matrix cores (k_split.h).
//
// A workgroup of eight (four) waves owns a 64 x 128 (32 x 128) output tile over the whole of K, a wave a 32 x 32 block of it.
// Per K block of 32 the threads load the fp32 rows of both operands (whole cache lines, two blocks ahead), split them once and
// lay the three parts out in LDS; a wave reads six 16-byte operands per six matrix instructions.  LDS is double-buffered, one
// workgroup barrier per K block.
// 1000 x 2000 x 400, one tile per CU: 20.3 us, of which 4.7 are matrix instructions, about as much are the vector
// instructions of the split, and the rest the phases between two barriers; the small fp32 tiles of k_gemm.hip take 31.
#include <type_traits>

#include "k_gemm_shared.h"
#include "k_split.h"

namespace {

constexpr int BK = 32;  // K block

template <int BM_, int BN_>
struct Shape {
    static constexpr int BM = BM_, BN = BN_;                    // output tile
    static constexpr int THREADS = BM / 32 * (BN / 32) * 64;
    static constexpr int PLANE_A = BM * BK, PLANE_B = BN * BK;  // bf16 elements of a part
    static constexpr int BUFFER = 3 * (PLANE_A + PLANE_B);
    static constexpr int STEP = THREADS / 8;                    // rows that the threads load together, 16 bytes each
    static constexpr int RA = BM / STEP, RB = BN / STEP;
};

// Element offset of K values 8 g .. 8 g + 7 of a row.  Rows are 64 bytes, four of them cross all LDS banks; the groups of
// rows 4 apart are permuted against each other, so that sixteen rows' reads of one g, and eight lanes' writes of a row, do not
// meet in a bank.
__device__ __forceinline__ int lds_at(int row, int g) { return row * BK + 8 * (g ^ ((row >> 2) & 3)); }

__device__ __forceinline__ void lds_barrier() {  // orders LDS traffic only: global loads stay in flight across it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// four K values of one row -> the three parts in LDS
template <bool LARGE>
__device__ __forceinline__ void store_split(float4 x, __bf16* plane, int stride, int row, int piece) {
    const Split2 lo = split2<LARGE>(x.x, x.y), hi = split2<LARGE>(x.z, x.w);
    __bf16* at = plane + lds_at(row, piece >> 1) + 4 * (piece & 1);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(at + q * stride) = make_uint2(lo.p[q], hi.p[q]);
}

template <int EPI, typename S>
__global__ __launch_bounds__(S::THREADS) void k_gemm_split_fwd(GemmArgs g) {
    constexpr int BM = S::BM, BN = S::BN, PLANE_A = S::PLANE_A, PLANE_B = S::PLANE_B, STEP = S::STEP, RA = S::RA, RB = S::RB;
    __shared__ __attribute__((aligned(16))) __bf16 lds[2][S::BUFFER];
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
    auto store = [&](int kb, Block& r, __bf16* buf) {
        if (kb * BK + BK > g.K) {  // (K is a multiple of 4)
            const bool in = kb * BK + 4 * piece < g.K;
#pragma unroll
            for (int q = 0; q < RA; ++q) r.a[q] = in ? r.a[q] : f4(0.f);
#pragma unroll
            for (int q = 0; q < RB; ++q) r.b[q] = in ? r.b[q] : f4(0.f);
        }
        float m = 0.f;
#pragma unroll
        for (int q = 0; q < RA; ++q) m = fmaxf(m, magnitude(r.a[q]));
#pragma unroll
        for (int q = 0; q < RB; ++q) m = fmaxf(m, magnitude(r.b[q]));
        auto put = [&](auto large) {
#pragma unroll
            for (int q = 0; q < RA; ++q) store_split<large.value>(r.a[q], buf, PLANE_A, row + STEP * q, piece);
#pragma unroll
            for (int q = 0; q < RB; ++q) store_split<large.value>(r.b[q], buf + 3 * PLANE_A, PLANE_B, row + STEP * q, piece);
        };
        if (__any(is_large(m))) put(std::true_type());
        else put(std::false_type());
    };
    floatx16 big = {}, small = {};
    auto multiply = [&](const __bf16* buf) {
        const int ra = wm + (lane & 31), rb = wn + (lane & 31);
#pragma unroll
        for (int s = 0; s < BK / 16; ++s) {
            Split8 a, b;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                a.p[q] = *reinterpret_cast<const bf16x8*>(buf + q * PLANE_A + lds_at(ra, 2 * s + (lane >> 5)));
                b.p[q] = *reinterpret_cast<const bf16x8*>(buf + 3 * PLANE_A + q * PLANE_B + lds_at(rb, 2 * s + (lane >> 5)));
            }
            mfma_split(a, b, big, small);
        }
    };
    const int nblk = (g.K + BK - 1) / BK, last = nblk - 1;
    Block r0 = issue(0), r1 = issue(min(1, last));
    for (int kb = 0; kb < nblk; kb += 2) {
        store(kb, r0, lds[0]);
        r0 = issue(min(kb + 2, last));
        lds_barrier();
        multiply(lds[0]);
        if (kb + 1 >= nblk) break;
        store(kb + 1, r1, lds[1]);
        r1 = issue(min(kb + 3, last));
        lds_barrier();
        multiply(lds[1]);
    }

    // ---- epilogue: register v of lane l holds element (8 (v/4) + 4 (l/32) + v%4, l%32) of the wave's block.  What it reads is
    // fetched before its first store.
    auto row_of = [&](int v) { return wm + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); };
    const int gn = n0 + wn + (lane & 31);
    float norm[16];
    if (EPI == EPI_L2_FWD) {
        const float cv = g.colv[c * g.s_colv + min(gn, g.N - 1)];
#pragma unroll
        for (int v = 0; v < 16; ++v) norm[v] = g.rowv[c * g.s_rowv + min(m0 + row_of(v), g.M - 1)] + cv;
    }
    float* C = g.C + c * g.sC;
    float loss = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int gm = m0 + row_of(v);
        const bool in = gm < g.M && gn < g.N;
        float s = big[v] + small[v], d = 0.f;
        if (EPI == EPI_L2_FWD) {
            d = sqrtf(fmaxf(norm[v] - 2.f * s, 0.f));
            s = g.gamma - d;
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
    }
}

template <int EPI, typename S>
void launch(kge_ctx* c, GemmArgs g, int chunks, hipStream_t st) {
    g.gx = (g.N + S::BN - 1) / S::BN;
    g.gy = (g.M + S::BM - 1) / S::BM;
    g.tiles = g.gx * g.gy * chunks;
    KGE_LAUNCH(c, (k_gemm_split_fwd<EPI, S>), dim3(8 * ((g.tiles + 7) / 8)), dim3(S::THREADS), 0, st, g);
}

// 32 rows per tile where a chunk has no more (1024 x 1500, D 400, chunks of 32: 51 us against 62 with 64 rows).
using Short = Shape<32, 128>;
using Tall = Shape<64, 128>;
bool short_chunk(int g) { return g <= Short::BM; }
template <int EPI>
void pick(kge_ctx* c, const GemmArgs& g, int chunks, hipStream_t st) {
    if (short_chunk(g.M)) launch<EPI, Short>(c, g, chunks, st);
    else launch<EPI, Tall>(c, g, chunks, st);
}

}  // namespace

int kge_gemm_split_blocks(int g, int k) {
    const int rows = short_chunk(g) ? Short::BM : Tall::BM, cols = Short::BN;
    static_assert(Short::BN == Tall::BN, "");
    return (g + rows - 1) / rows * ((k + cols - 1) / cols) * (rows / 32 * (cols / 32));
}

void kge_gemm_split_forward(kge_ctx* c, const void* args, int epi, int chunks, hipStream_t st) {
    const GemmArgs& g = *static_cast<const GemmArgs*>(args);
    if (epi == EPI_L2_FWD) pick<EPI_L2_FWD>(c, g, chunks, st);
    else pick<EPI_PLAIN>(c, g, chunks, st);
}
