// TransR (Table 1 of the paper): f(h, r, t) = gamma - |M_r h + r - M_r t|_2^2.  A relation row holds the translation r
// (D numbers) followed by the D x D projection M_r, row by row.
//
// With a the entity that is kept, x the one that is replaced (the true one for the positive, a corrupting one for a
// negative) and sigma = +1 (tail corrupted) or -1 (head corrupted):
//     o_i = M_i a_i + sigma r_i ,    P(x) = M_i x ,    f = gamma - |o_i - P(x)|^2
// so a positive's negatives need the chunk's corrupting rows projected with the positive's own matrix.  Positives of one
// chunk that share a relation share these projections, and what flows back through them adds up before it is
// multiplied: the unit of work is an ITEM, a (chunk, relation) that occurs in the mini-batch, with its positives.  The
// arrays per positive (o, p, gradients, scores, coefficients) are in the order of the items' positives ("members"), so
// that an item's rows are contiguous; what a caller sees is put back into the order of the mini-batch where it is stored.
//   (k_gather)        the items of every chunk (k_transr_items.h), beside the corrupting rows and the order of the keys
//   k_transr_phi      o_i, p_i = M_i c_i: an item's a and c rows times M^T; the positive's score and logistic-loss terms
// then, where W needs no loss kernel (logistic loss, uniform weights, up to 1024 scores per row) and rows have up to 128 floats:
//   k_transr_project_units  (k_transr_unit.h) scores, W, V and the corrupting rows' gradients in one pass over the UNITS, the blocks
//                     of up to 32 positives of an item
//   k_transr_go       dL/do_i, dL/dp_i and the gradient of the translation from their parts
//   k_transr_mgrad    dL/dM of a unit: V_t^T N_c + sum over its positives of dL/do a^T + dL/dp c^T, one product whose K range is
//                     the corrupting rows and the positives; beside it M^T dL/do_i, M^T dL/dp_i
// and otherwise
//   k_transr_project  P_t = N_c M_t^T, and in its epilogue S_ij = gamma - |o_i - P_tj|^2 for the item's positives (or W = dL/df-)
//   (k_loss)          W
//   k_transr_dp       V_tj = sum over the item's positives of 2 W_ij (o_i - P_tj); dL/do_i = - sum_j of the same terms
//                     - 2 cpos (o - p), dL/dp_i = 2 cpos (o - p), gradient of the translation (k_transr_go ends these for
//                     items of few positives)
//   k_transr_back     sum over a chunk's items of V_t M_t (partial over ranges of items); M^T dL/do_i, M^T dL/dp_i
//   k_transr_mgrad    dL/dM of an item
// and in the end
//   k_transr_update   duplicate reduction and Adagrad for the relation rows [r | M] (Sec. 3.1 step 4); the partial sums
//                     of the corrupting rows' gradients
// The products (but for k_transr_unit.h's) run on v_mfma_f32_16x16x4_f32, those of k_transr_back and k_transr_mgrad of longer rows on
// the bf16 matrix cores: a workgroup owns 64 rows x up to 128 columns (whole matrices at D <= 128),
// K in blocks of 32 staged in LDS for its four waves (16 rows each), the next block's global loads in flight while one is
// multiplied.  (128 rows per workgroup were measured: equal or slower, half as many waves fit a SIMD.)  All sums have a
// fixed order.
// FB15k-sized (b 1024, g 128, k 256, D 100; 667 items of the 1024 positives): 190 us per step; 250 with projection, V M and M^T dL/do
// in launches of their own, 292 with all products in fp32 and V in a launch too (450 with three products per positive on 32x32 tiles).
#include <type_traits>

#include "k_gemm_shared.h"
#include "k_transr_items.h"
#include "k_weights.h"

namespace {

constexpr int RT = 256;
constexpr int BM = 64, BN = 128, BK = 32;  // rows, most columns, K per staged block
constexpr int KP = 36;                     // pitch of a staged [row][k] block: 16-byte reads without bank conflicts
constexpr int AP = BM + 4, BP = BN + 4;    // pitches of staged [k][row] blocks: 4 * pitch = 16 mod 64 banks
constexpr int A_FLOATS = BM * KP > BK * AP ? BM * KP : BK * AP, B_FLOATS = BN * KP > BK * BP ? BN * KP : BK * BP;
constexpr int PB = TRANSR_PB;              // positives per block of an item's positives
constexpr int DP_FEW = 16;                 // items of at most so many positives: V and dL/do positive by positive
static_assert(DP_FEW <= PB, "such an item is one block");

typedef double doublex4 __attribute__((ext_vector_type(4)));

struct TransrArgs {
    const float* E;
    const float* R;
    StepIds ids;
    int b, D, k, g, ld_s, max_items, max_pblocks;  // (the last two per chunk)
    int64_t n_ent, n_rel, rel_dim;
    float gamma, wk;
    int out_w;       // project: store W = dL/df- instead of the score
    int train;       // project: keep the projections, scores in the order of the members; phi: likewise
    int segments;    // back, unit: ranges of a chunk's items (units)
    int units;       // k_transr_project_units runs, or has run: gradients of the positives in parts of 16 rows, V and matrix gradients by unit
    int unit_rows;   // unit: corrupting rows per workgroup
    TransrGroups q;
    float* O;        // [b x D]      o
    float* PP;       // [b x D]      p, then dL/dp
    float* P;        // [b x k x D]  projections of item slot t
    float* V;        // [b x k x D]  dL/dP summed over the item's positives
    const float* N;  // [C*k x D]    corrupting rows
    float* S;        // [b x ld_s]   scores, then W
    float* GO;       // [b x D]      dL/do
    float* GOp;      // [ceil(k / 64)][b x D] partial sums of it (items of few positives)
    float* fpos;
    float* pos_out;
    float* cpos;
    float* row_loss;
    float* loss_part;
    float* Gent;     // gradient rows in key order: heads | tails | corrupting rows
    float* Gr;       // [b x D]      gradient of the translation, in the order of the mini-batch
    float* GM;       // [b x D x D]  gradient of the matrix, per item slot
    float* back_part;  // [segments][C*k x D]
};

// ---------------------------------------------------------------------------------------------------------------
// The product core.  Thread tid stages, per block of 32 values of K, pieces of 16 bytes:
//   [row][k] operands: row tid / 8 + 32 it, k 4 (tid % 8) ..      (A: 2 pieces, B: 4)
//   [k][row] operands: A: k tid / 16 + 16 it, row 4 (tid % 16) ..  B: k tid / 32 + 8 it, row 4 (tid % 32) ..
// load_a / load_b(run, block, piece registers) ask for them; mask_a / mask_b put zeros where k is outside the product, a
// block later, when they go to LDS (a select right behind the load would wait for it).  Rows outside only reach outputs
// that are not stored, and read something valid.  No branch stands between the loads of a block, and none between the LDS
// reads and matrix instructions of one (the number of column tiles NT is a template argument).
// F64: operands in 32 bits, products and sums in 64.
template <int NT, bool F64 = false>
struct Tile {
    typedef typename std::conditional<F64, double, float>::type Sum;
    typedef typename std::conditional<F64, doublex4, floatx4>::type Acc;
    float* As;
    float* Bs;
    Acc acc[NT];
    Sum a_sum;  // ASUM: sum over K of the A values of row lane % 16 of the wave's sixteen (complete in every lane)
    int wave, lane;
    bool active;  // the wave has rows
    __device__ __forceinline__ int row16(int v) const { return F64 ? (lane >> 4) + 4 * v : 4 * (lane >> 4) + v; }
    __device__ __forceinline__ int row(int v) const { return 16 * wave + row16(v); }  // of accumulator v
    __device__ __forceinline__ Sum a_sum_of(int v) const { return __shfl(a_sum, row16(v), 64); }
};

// Waves take the groups of 16 rows in an order that changes from workgroup to workgroup, so that the SIMDs of a CU get about
// the same number where there are fewer than four.
__device__ __forceinline__ int row_wave() { return __builtin_amdgcn_readfirstlane(((threadIdx.x >> 6) + blockIdx.x) & 3); }
template <int NT, bool F64>
__device__ __forceinline__ void tile_init(Tile<NT, F64>& t, float* As, float* Bs, int rows) {
    t.As = As; t.Bs = Bs;
    t.wave = row_wave(); t.lane = threadIdx.x & 63;
    t.active = __builtin_amdgcn_readfirstlane(16 * t.wave < rows);
    t.a_sum = 0.f;
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) t.acc[ct] = typename Tile<NT, F64>::Acc{0, 0, 0, 0};
}

// 16 values of K (from s16 on) of a staged block
template <bool A_KC, bool B_KC, bool ASUM, int NT, bool F64>
__device__ __forceinline__ void tile_mma(Tile<NT, F64>& t, int s16) {
    const int r16 = t.lane & 15, kk = s16 + 4 * (t.lane >> 4), row = 16 * t.wave + r16;
    float fa[4];
    if (A_KC) {
        const float4 v = ld4(t.As + row * KP + kk);
        fa[0] = v.x; fa[1] = v.y; fa[2] = v.z; fa[3] = v.w;
    } else {
#pragma unroll
        for (int x = 0; x < 4; ++x) fa[x] = t.As[(kk + x) * AP + row];
    }
    typedef typename Tile<NT, F64>::Sum Sum;
    if (ASUM) t.a_sum += ((Sum)fa[0] + fa[1]) + ((Sum)fa[2] + fa[3]);
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
        float fb[4];
        if (B_KC) {
            const float4 v = ld4(t.Bs + (16 * ct + r16) * KP + kk);
            fb[0] = v.x; fb[1] = v.y; fb[2] = v.z; fb[3] = v.w;
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x) fb[x] = t.Bs[(kk + x) * BP + 16 * ct + r16];
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            if constexpr (F64) t.acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[x], fb[x], t.acc[ct], 0, 0, 0);
            else t.acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[x], fb[x], t.acc[ct], 0, 0, 0);
        }
    }
}

// The product over `runs` consecutive ranges of K values each; masks apply to the last block of a run.
template <bool A_KC, bool B_KC, bool ASUM, int NT, bool F64, class LoadA, class MaskA, class LoadB, class MaskB>
__device__ __forceinline__ void tile_run(Tile<NT, F64>& t, int K, int runs, LoadA load_a, MaskA mask_a, LoadB load_b, MaskB mask_b) {
    constexpr int NB = B_KC ? (NT + 1) / 2 : 4;  // pieces of B that hold columns of the tile
    const int tid = threadIdx.x;
    const int bpr = (K + BK - 1) / BK, nblk = bpr * runs;
    const bool odd = K - BK * (bpr - 1) <= 16;  // the last block of a run is at most 16 values
    float4 ra[2], rb[4];
    float* sa = A_KC ? t.As + tid / 8 * KP + 4 * (tid % 8) : t.As + tid / 16 * AP + 4 * (tid % 16);
    float* sb = B_KC ? t.Bs + tid / 8 * KP + 4 * (tid % 8) : t.Bs + tid / 32 * BP + 4 * (tid % 32);
    int run = 0, kb = 0;  // of the block that is loaded
    if (nblk > 0) { load_a(0, 0, ra); load_b(0, 0, rb); }
    for (int blk = 0; blk < nblk; ++blk) {
        const bool tail = kb == bpr - 1;
        __syncthreads();  // the block before has been read
        if (tail) { mask_a(kb, ra); mask_b(kb, rb); }
#pragma unroll
        for (int it = 0; it < 2; ++it) st4(sa + it * (A_KC ? 32 * KP : 16 * AP), ra[it]);
#pragma unroll
        for (int it = 0; it < NB; ++it) st4(sb + it * (B_KC ? 32 * KP : 8 * BP), rb[it]);
        __syncthreads();
        if (tail) { kb = 0; ++run; } else { ++kb; }
        if (blk + 1 < nblk) { load_a(run, kb, ra); load_b(run, kb, rb); }
        if (t.active) {
            const int ns = tail && odd ? 1 : 2;
#pragma unroll 1
            for (int s = 0; s < ns; ++s) tile_mma<A_KC, B_KC, ASUM>(t, 16 * s);
        }
    }
    if (ASUM) {
        t.a_sum += __shfl_xor(t.a_sum, 16, 64);
        t.a_sum += __shfl_xor(t.a_sum, 32, 64);
    }
}

// pieces of a [row][k] operand whose rows of K floats start at p[it]
template <int N>
__device__ __forceinline__ void load_kc(const float* const (&p)[N], int K, int blk, float4* r) {
    const int k = BK * blk + 4 * (threadIdx.x % 8);
#pragma unroll
    for (int it = 0; it < N; ++it) r[it] = ld4(p[it] + (k < K ? k : 0));
}
template <int N>
__device__ __forceinline__ void mask_kc(int K, int blk, float4* r) {
    const bool out = BK * blk + 4 * (int)(threadIdx.x % 8) >= K;
#pragma unroll
    for (int it = 0; it < N; ++it) r[it] = out ? f4(0.f) : r[it];
}
// [k][row] operand with rows of `ld` floats from p on (the thread's column included): k of piece it is BK blk + k0 + step it
template <int N>
__device__ __forceinline__ void load_mc(const float* p, int64_t ld, int K, int blk, int k0, int step, float4* r) {
#pragma unroll
    for (int it = 0; it < N; ++it) r[it] = ld4(p + min(BK * blk + k0 + step * it, K - 1) * ld);
}
template <int N>
__device__ __forceinline__ void mask_mc(int K, int blk, int k0, int step, float4* r) {
#pragma unroll
    for (int it = 0; it < N; ++it) r[it] = BK * blk + k0 + step * it >= K ? f4(0.f) : r[it];
}

// ---------------------------------------------------------------------------------------------------------------
// Products whose B is stored with K along its rows, on the bf16 matrix cores, operands in three parts (k_split.h): 96 matrix
// cycles per 16 x 16 x 32 instead of 256.  A wave's sixteen rows of A are its own, so they go from memory to registers as the
// instruction wants them (lane: row lane % 16, eight values of K from 8 (lane / 16) on) and are split there; B is split once
// on its way to LDS, [column][k], 80 bytes per column with the 16-byte groups permuted by column / 16, so that neither the
// reads of 16 columns nor the transposing writes (columns four apart) pile up on a few banks.
// From SPLIT_FROM column tiles on, where the matrix instructions outweigh what splitting adds to the chain of a K block
// (k_transr_back, k_transr_mgrad; us per step, fp32 -> split): D 100 FB15k-sized 290 -> 270, D 124 k 500 340 -> 287, D 400 401 ->
// 370, D 96 97.3 -> 93.0; D 64 62.5 -> 70.3, D 48 153.5 -> 158.5.  The projections (B with K along its columns) measured the
// same at D 100 and slower elsewhere (D 400: 123 -> 147).  Three workgroups per CU: held to four they spill, two are slower
// (FB15k-sized 239 against 268).  Error against 64 bits of the entities' gradients 1.9e-7 -> 0.7e-7, matrices 0.9e-7 -> 0.6e-7.
constexpr int SPLIT_FROM = 5;
constexpr int SP = 40;  // bf16 per column
__device__ __forceinline__ int split_at(int col, int group) { return col * SP + 8 * (group ^ ((col >> 4) & 3)); }

template <int NT>
struct SplitTile {
    floatx4 big[NT], acc[NT];  // (acc: the small products, after split_run the sum)
    int wave, lane;
    bool active;  // the wave has rows
    __device__ __forceinline__ int row16(int v) const { return 4 * (lane >> 4) + v; }
    __device__ __forceinline__ int row(int v) const { return 16 * wave + row16(v); }  // of accumulator v
    __device__ __forceinline__ int a_row() const { return 16 * wave + (lane & 15); }  // of A
    __device__ __forceinline__ int a_k() const { return 8 * (lane >> 4); }
};
template <int NT>
__device__ __forceinline__ void split_init(SplitTile<NT>& t, int rows) {
    t.wave = row_wave(); t.lane = threadIdx.x & 63;
    t.active = __builtin_amdgcn_readfirstlane(16 * t.wave < rows);
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) t.big[ct] = t.acc[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
}

// A thread's piece of B, K values 4 (tid / 32) .. of columns 4 (tid % 32) .., transposed on the way to LDS
template <bool LARGE>
__device__ __forceinline__ void split_store(uint16_t* Bs, int stride, int cols, const float4 (&r)[4]) {
    const int tid = threadIdx.x, k = 4 * (tid / 32);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int col = 4 * (tid % 32) + it;
        if (col >= cols) continue;
        auto at_col = [&](const float4& v) { return it == 0 ? v.x : it == 1 ? v.y : it == 2 ? v.z : v.w; };
        const Split2 lo = split2<LARGE>(at_col(r[0]), at_col(r[1])), hi = split2<LARGE>(at_col(r[2]), at_col(r[3]));
        uint16_t* at = Bs + split_at(col, k >> 3) + (k & 4);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(at + q * stride) = make_uint2(lo.p[q], hi.p[q]);
    }
}
template <bool LARGE>
__device__ __forceinline__ Split8 split_row(const float4& x, const float4& y) {
    const Split2 s[4] = {split2<LARGE>(x.x, x.y), split2<LARGE>(x.z, x.w), split2<LARGE>(y.x, y.y), split2<LARGE>(y.z, y.w)};
    Split8 r;
#pragma unroll
    for (int q = 0; q < 3; ++q) r.p[q] = __builtin_bit_cast(bf16x8, make_uint4(s[0].p[q], s[1].p[q], s[2].p[q], s[3].p[q]));
    return r;
}

// Bs: uint16_t [3][16 NT][SP].  load_a(run, block, two pieces): A's row a_row(), K values a_k() .. a_k() + 7 of the block.
template <int NT, class LoadA, class MaskA, class LoadB, class MaskB>
__device__ __forceinline__ void split_run(SplitTile<NT>& t, uint16_t* Bs, int K, int runs, LoadA load_a, MaskA mask_a, LoadB load_b, MaskB mask_b) {
    constexpr int STRIDE = 16 * NT * SP;
    const int bpr = (K + BK - 1) / BK, nblk = bpr * runs;
    float4 ra[2], rb[4];
    int run = 0, kb = 0;  // of the block that is loaded
    if (nblk > 0) { load_a(0, 0, ra); load_b(0, 0, rb); }
    for (int blk = 0; blk < nblk; ++blk) {
        if (kb == bpr - 1) { mask_a(kb, ra); mask_b(kb, rb); }
        float m = 0.f, ma = fmaxf(magnitude(ra[0]), magnitude(ra[1]));
#pragma unroll
        for (int it = 0; it < 4; ++it) m = fmaxf(m, magnitude(rb[it]));
        Split8 a;
        if (__any(is_large(ma))) a = split_row<true>(ra[0], ra[1]);
        else a = split_row<false>(ra[0], ra[1]);
        __syncthreads();  // the block before has been read
        if (__any(is_large(m))) split_store<true>(Bs, STRIDE, 16 * NT, rb);
        else split_store<false>(Bs, STRIDE, 16 * NT, rb);
        __syncthreads();
        if (kb == bpr - 1) { kb = 0; ++run; } else { ++kb; }
        if (blk + 1 < nblk) { load_a(run, kb, ra); load_b(run, kb, rb); }
        if (t.active) {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                const uint16_t* p = Bs + split_at(16 * ct + (t.lane & 15), t.lane >> 4);
                Split8 b;
#pragma unroll
                for (int q = 0; q < 3; ++q) b.p[q] = *reinterpret_cast<const bf16x8*>(p + q * STRIDE);
                mfma_split(a, b, t.big[ct], t.acc[ct]);
            }
        }
    }
}
template <int NT>
__device__ __forceinline__ void split_sum(SplitTile<NT>& t) {
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) t.acc[ct] += t.big[ct];
}
// a row of A whose K floats start at p
__device__ __forceinline__ void load_row(const float* p, int k, int K, float4 (&r)[2]) {
    r[0] = ld4(p + (k < K ? k : 0));
    r[1] = ld4(p + (k + 4 < K ? k + 4 : 0));
}
__device__ __forceinline__ void mask_row(int k, int K, float4 (&r)[2]) {
    r[0] = k < K ? r[0] : f4(0.f);
    r[1] = k + 4 < K ? r[1] : f4(0.f);
}

// x of the lane that control word CTRL names (within a row of 16 lanes: vector ALU moves, no LDS)
template <int CTRL> __device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_ROR8 = 0x128;
__device__ __forceinline__ float sum16(float x) {  // over the 16 lanes of a row, in every lane
    x += dpp<DPP_ROR8>(x);
    x += dpp<DPP_HALF_MIRROR>(x);  // (lane i and 7 - i: what they lack of each other's quad the next two steps add)
    x += dpp<DPP_XOR2>(x);
    x += dpp<DPP_XOR1>(x);
    return x;
}
// sums over 16 lanes of four values; lane (of the 16) with bits 3, 2 = (h1, h2) gets value 2 h1 + h2
__device__ __forceinline__ float sum16x4(const float (&s)[4]) {
    const bool h1 = threadIdx.x & 8, h2 = threadIdx.x & 4;
    float x = h1 ? s[2] : s[0], y = h1 ? s[3] : s[1];
    x += dpp<DPP_ROR8>(h1 ? s[0] : s[2]);
    y += dpp<DPP_ROR8>(h1 ? s[1] : s[3]);
    float z = h2 ? y : x;
    z += dpp<DPP_HALF_MIRROR>(h2 ? x : y);
    z += dpp<DPP_XOR2>(z);
    z += dpp<DPP_XOR1>(z);
    return z;
}

// Workgroup -> (item or block of an item's positives, tile): the tiles of an item run on one XCD (workgroups are dealt to
// them round-robin) and share its operands there.
__device__ __forceinline__ int unit_of_block(int block, int tiles, int& tile) {
    const int xcd = block & 7, n = block >> 3;
    tile = n % tiles;
    return n / tiles * 8 + xcd;
}
int unit_blocks(int units, int tiles) { return (units + 7) / 8 * 8 * tiles; }
int item_blocks(const TransrArgs& a, int tiles) { return unit_blocks(a.b / a.g * a.max_items, tiles); }
int pblock_blocks(const TransrArgs& a, int tiles) { return unit_blocks(a.b / a.g * a.max_pblocks, tiles); }
// The record of the unit and the number of units in its chunk are asked for together.
__device__ __forceinline__ bool item_of(const TransrArgs& a, int unit, int& c, int& slot, TransrItem& item) {
    c = unit / a.max_items;
    const int idx = unit - c * a.max_items;
    slot = c * a.g + idx;
    if (c * a.g >= a.b) return false;
    item = a.q.items[slot];
    return idx < a.q.n_items[c];
}
__device__ __forceinline__ bool pblock_of(const TransrArgs& a, int unit, int& c, TransrBlock& blk) {
    c = unit / a.max_pblocks;
    const int e = unit - c * a.max_pblocks;
    if (c * a.g >= a.b) return false;
    blk = a.q.pblocks[(int64_t)c * a.max_pblocks + e];
    return e < a.q.n_pblocks[c];
}

// a unit as an item of its own
__device__ __forceinline__ bool unit_item_of(const TransrArgs& a, int unit, int& c, int& slot, TransrItem& item) {
    TransrBlock blk;
    if (!pblock_of(a, unit, c, blk)) return false;
    slot = c * a.g + unit - c * a.max_pblocks;
    item = {blk.rel, blk.off, blk.n};
    return true;
}

__device__ __forceinline__ void lds_barrier() {  // orders LDS traffic only: global loads stay in flight across it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace
#include "k_transr_unit.h"
namespace {

// Rows 2 m and 2 m + 1 of the product: a and c of the block's m-th positive.
template <int NT>
__global__ __launch_bounds__(RT) void k_transr_phi(TransrArgs a) {
    __shared__ __attribute__((aligned(16))) float As[A_FLOATS], Bs[B_FLOATS];
    const int D = a.D, tid = threadIdx.x;
    int c;
    TransrBlock blk;
    if (!pblock_of(a, blockIdx.x, c, blk)) return;
    const int n = blk.n;
    const StepView sv = step_view(a.ids);
    const bool head = sv.side == KGE_NEG_HEAD;
    const float* Rr = a.R + (int64_t)blk.rel * a.rel_dim;
    const float* M = Rr + D;
    const float* pa[2];
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int row = min(tid / 8 + 32 * it, 2 * n - 1), i = a.q.members[blk.off + row / 2];
        // even rows: the kept entity, odd rows: the replaced one
        const int64_t id = clamp_id((head == (bool)(row & 1)) ? sv.h[i] : sv.t[i], a.n_ent);
        pa[it] = a.E + id * D;
        if (tid % 8 == 0 && row == tid / 8 + 32 * it) a.q.ent[2 * blk.off + row] = (uint32_t)id;
    }
    if (a.units && tid < n) a.q.unit_of[a.q.members[blk.off + tid]] = tid > 0 ? -1 : c * a.g + (int)blockIdx.x - c * a.max_pblocks;
    const float sigma = head ? -1.f : 1.f;
    const int l16 = tid & 15, quad = (tid & 63) >> 4;
    float ss[2] = {0.f, 0.f};
    for (int n0 = 0; n0 < D; n0 += BN) {
        Tile<NT> t;
        tile_init(t, As, Bs, 2 * n);
        const float* pb[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) pb[it] = M + (int64_t)min(n0 + tid / 8 + 32 * it, D - 1) * D;
        float rr[NT];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) rr[ct] = sigma * Rr[min(n0 + 16 * ct + l16, D - 1)];
        tile_run<true, true, false>(t, D, 1, [&](int, int kb, float4* r) { load_kc<2>(pa, D, kb, r); },
                                    [&](int kb, float4* r) { mask_kc<2>(D, kb, r); },
                                    [&](int, int kb, float4* r) { load_kc<4>(pb, D, kb, r); },
                                    [&](int kb, float4* r) { mask_kc<4>(D, kb, r); });
        if (!t.active) continue;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int d = n0 + 16 * ct + l16;
            if (d < D) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int m = 8 * t.wave + 2 * quad + h;
                    const float o = t.acc[ct][2 * h] + rr[ct], p = t.acc[ct][2 * h + 1];
                    ss[h] += (o - p) * (o - p);
                    if (m < n) {
                        const int64_t at = (int64_t)(blk.off + m) * D + d;
                        a.O[at] = o;
                        a.PP[at] = p;
                    }
                }
            }
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float s = sum16(ss[h]);
        const int m = 8 * row_wave() + 2 * quad + h;
        if (l16 == 0 && m < n) {
            const int q = blk.off + m, i = a.train ? q : a.q.members[q];
            const float f = a.gamma - s;
            a.fpos[i] = f;
            if (a.pos_out) a.pos_out[i] = f;
            // positive part of the logistic loss (Sec. 2, y = +1) and its derivative
            const float invb = 1.f / (float)a.b;
            const float x = expf(-fabsf(f));
            a.row_loss[i] = (fmaxf(-f, 0.f) + log1pf(x)) * invb;
            a.cpos[i] = -((f >= 0.f ? x : 1.f) / (1.f + x)) * invb;
        }
    }
}

// 64 corrupting rows x a block of an item's positives: projections, then the scores of the positives against them.  (An
// item of more than 32 positives is projected once per block: at that size the scores are the larger part of the work.)
template <int NT>
__global__ __launch_bounds__(RT, 4) void k_transr_project(TransrArgs a, int blocks) {
    __shared__ __attribute__((aligned(16))) float As[A_FLOATS], Bs[B_FLOATS];
    const int tiles = (a.k + BM - 1) / BM, D = a.D, tid = threadIdx.x;
    int c, tile;
    TransrBlock blk;
    float loss = 0.f;
    const int block = flat_block();
    if (block >= blocks) return;
    const int unit = unit_of_block(block, tiles, tile);
    if (pblock_of(a, unit, c, blk)) {
        const int j0 = tile * BM, rows = min(BM, a.k - j0), n = blk.n;
        const float* M = a.R + (int64_t)blk.rel * a.rel_dim + D;
        const float* N = a.N + ((int64_t)c * a.k + j0) * D;
        float* P = a.P + ((int64_t)blk.slot * a.k + j0) * D;
        const float* pa[2];
#pragma unroll
        for (int it = 0; it < 2; ++it) pa[it] = N + (int64_t)min(tid / 8 + 32 * it, rows - 1) * D;
        const int l16 = tid & 15, q = ((tid >> 2) & 1) + 2 * ((tid >> 3) & 1);  // accumulator row this lane ends up with
        for (int n0 = 0; n0 < D; n0 += BN) {
            Tile<NT> t;
            tile_init(t, As, Bs, rows);
            const float* pb[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) pb[it] = M + (int64_t)min(n0 + tid / 8 + 32 * it, D - 1) * D;
            tile_run<true, true, false>(t, D, 1, [&](int, int kb, float4* r) { load_kc<2>(pa, D, kb, r); },
                                        [&](int kb, float4* r) { mask_kc<2>(D, kb, r); },
                                        [&](int, int kb, float4* r) { load_kc<4>(pb, D, kb, r); },
                                        [&](int kb, float4* r) { mask_kc<4>(D, kb, r); });
            // the o rows of the block, where the matrix was (zeros past column D)
            float4 ro[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int d = n0 + 4 * (tid % 32);
                ro[it] = d < D ? ld4(a.O + (int64_t)(blk.off + min(tid / 32 + 8 * it, n - 1)) * D + d) : f4(0.f);
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < 4; ++it) st4(Bs + (tid / 32 + 8 * it) * BN + 4 * (tid % 32), ro[it]);
            __syncthreads();
            if (!t.active) continue;
            const bool store_p = a.train && blk.first == 0;
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                const int d = n0 + 16 * ct + l16;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (d >= D) t.acc[ct][v] = 0.f;
                    else if (store_p && t.row(v) < rows) P[(int64_t)t.row(v) * D + d] = t.acc[ct][v];
                }
            }
            // four positives per round, so that every lane has a score to finish: positive m0 + lane % 4, row q
            const int x = tid & 3, j = t.row(q);
            for (int m0 = 0; m0 < n; m0 += 4) {
                float r[4];
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    if (m0 + y >= n) {
                        r[y] = 0.f;
                        continue;
                    }
                    const float* po = Bs + (m0 + y) * BN + l16;
                    float ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ct = 0; ct < NT; ++ct) {
                        const float o = po[16 * ct];
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float d = o - t.acc[ct][v];
                            ss[v] = fmaf(d, d, ss[v]);
                        }
                    }
                    r[y] = sum16x4(ss);
                }
                if (m0 + x >= n || j >= rows) continue;
                float s = x == 0 ? r[0] : x == 1 ? r[1] : x == 2 ? r[2] : r[3];
                const int m = blk.off + m0 + x;
                float* ps = a.S + (int64_t)(a.train ? m : a.q.members[m]) * a.ld_s + j0 + j;
                if (n0 > 0) s += *ps;  // what the columns before contributed
                if (n0 + BN >= D) {
                    s = a.gamma - s;
                    if (a.out_w) s = w_and_loss<true>(s, a.wk, loss);
                }
                *ps = s;
            }
        }
    }
    if (!a.out_w) return;
    __shared__ float part[RT / 64];
    loss = wave_sum(loss);
    if ((tid & 63) == 0) part[tid >> 6] = loss;
    __syncthreads();
    if (tid == 0) a.loss_part[block] = (part[0] + part[1] + part[2] + part[3]) * a.wk;
}

// Items of at most DP_FEW positives: the sums over an item's positives and over the corrupting rows on the vector ALUs,
// both while a row of P is in registers (32 us for the FB15k-sized step, 130 MB of rows; two products took 67, their
// tiles of sixteen rows nearly empty); others: two products.
constexpr int MB = 4, DR = 8;
constexpr int DN = 64;  // columns of a tile of those products

// 64 corrupting rows of an item.  Thread (group, 16 bytes of the row), DR rows at a time in registers with their sums over
// the item's positives, which come in batches of MB: the sums for dL/do stay in registers too and meet in LDS in group order.
__device__ void dp_few(const TransrArgs& a, int slot, int tile, const TransrItem& item, float4 (*part)[RT], float (*W2)[BM]) {
    const int D = a.D, tid = threadIdx.x, lanes = D / 4, groups = RT / lanes, n = item.n;
    const int j0 = tile * BM, rows = min(BM, a.k - j0), grp = tid / lanes, v = tid % lanes;
    const bool act = grp < groups;
    const int64_t base = ((int64_t)slot * a.k + j0) * D + 4 * v;
    const float* O = a.O + (int64_t)item.off * D + 4 * v;
    const int wm = tid / BM, wj = tid % BM;
    const float* W = a.S + (int64_t)item.off * a.ld_s + j0 + min(wj, rows - 1);
    for (int r0 = 0; r0 < rows; r0 += DR * groups) {
        float4 p[DR], s[DR];
#pragma unroll
        for (int u = 0; u < DR; ++u) {
            p[u] = ld4(a.P + base + (int64_t)min(r0 + (act ? grp : 0) + u * groups, rows - 1) * D);
            s[u] = f4(0.f);
        }
        for (int m0 = 0; m0 < n; m0 += MB) {
            const int mn = min(MB, n - m0);
            float4 o[MB], go[MB];
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                o[m] = ld4(O + (int64_t)min(m0 + m, n - 1) * D);
                go[m] = f4(0.f);
            }
            const float w2 = 2.f * W[(int64_t)min(m0 + wm, n - 1) * a.ld_s];
            __syncthreads();
            W2[wm][wj] = wm < mn && wj < rows ? w2 : 0.f;  // (rows and positives that do not exist add nothing)
            __syncthreads();
#pragma unroll
            for (int u = 0; u < DR; ++u) {
                const int j = r0 + grp + u * groups;
                if (act && j < rows) {
#pragma unroll
                    for (int m = 0; m < MB; ++m) {
                        const float w = W2[m][j];
                        const float4 x = make_float4(w * (o[m].x - p[u].x), w * (o[m].y - p[u].y), w * (o[m].z - p[u].z), w * (o[m].w - p[u].w));
                        s[u].x += x.x; s[u].y += x.y; s[u].z += x.z; s[u].w += x.w;
                        go[m].x -= x.x; go[m].y -= x.y; go[m].z -= x.z; go[m].w -= x.w;
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < MB; ++m) part[m][tid] = go[m];
            __syncthreads();
            for (int e = tid; e < mn * lanes; e += RT) {
                const int m = e / lanes, x = e % lanes;
                float4 t = part[m][x];
                for (int g2 = 1; g2 < groups; ++g2) {
                    const float4 q = part[m][g2 * lanes + x];
                    t.x += q.x; t.y += q.y; t.z += q.z; t.w += q.w;
                }
                float* dst = a.GOp + ((int64_t)tile * a.b + item.off + m0 + m) * D + 4 * x;
                if (r0 > 0) {
                    const float4 q = ld4(dst);
                    t.x += q.x; t.y += q.y; t.z += q.z; t.w += q.w;
                }
                st4(dst, t);
            }
        }
#pragma unroll
        for (int u = 0; u < DR; ++u) {
            const int j = r0 + grp + u * groups;
            if (act && j < rows) st4(a.V + base + (int64_t)j * D, s[u]);
        }
    }
}

// The first workgroups: the gradients of a block of the positives of an item of many x 64 columns, K over the corrupting
// rows; the others: V of 64 corrupting rows of an item (of many: K over the item's positives, 64 columns at a time).
//     V = 2 (W^T O - colsum(W) P) ,   dL/do = 2 (W P - rowsum(W) o)
// These differences cancel where o is close to P, so both products are formed in 64 bits (v_mfma_f64_16x16x4_f64, half the
// rate) and what is left is the rounding of the result.  Items of 17 to 97 positives, rows a hundredth of their length
// apart, error of the entities' gradients: products in 32 bits 0.7 to 2.0e-4, in 64 bits 1.8 to 2.4e-7 (sums of 2 W (o - P),
// positive by positive, 1.8 to 2.9e-7).  64 columns, so that the accumulators take the registers that 128 take in 32 bits:
// dp_few needs its three waves per SIMD.  Per step, 32 -> 64 bits: FB15k-sized 279 -> 281 us, b 1024, g 1024, k 1024, D 128,
// 2 relations 347 -> 360, b 1024, g 128, k 256, D 100, 2 relations 134.7 both.
template <int NT>
__global__ __launch_bounds__(RT) void k_transr_dp(TransrArgs a, int go_blocks, int blocks) {
    __shared__ __attribute__((aligned(16))) float lds[A_FLOATS + B_FLOATS];
    float* As = lds;
    float* Bs = lds + A_FLOATS;
    static_assert(sizeof(float4) * MB * RT + sizeof(float) * MB * BM <= sizeof(lds), "");
    const int D = a.D, tid = threadIdx.x, l16 = tid & 15, block = flat_block();
    int c;
    if (block >= blocks) return;
    if (block >= go_blocks) {
        int slot, tile;
        TransrItem item;
        const int tiles = (a.k + BM - 1) / BM;
        if (!item_of(a, unit_of_block(block - go_blocks, tiles, tile), c, slot, item)) return;
        const int j0 = tile * BM, rows = min(BM, a.k - j0), n = item.n;
        if (n <= DP_FEW) {
            dp_few(a, slot, tile, item, reinterpret_cast<float4(*)[RT]>(lds), reinterpret_cast<float(*)[BM]>(lds + 4 * MB * RT));
            return;
        }
        const int ja = 4 * (tid % 16);
        const float* W = a.S + (int64_t)item.off * a.ld_s + j0 + (ja < rows ? ja : 0);
        for (int n0 = 0; n0 < D; n0 += DN) {
            const int db = n0 + 4 * (tid % 32);
            const float* O = a.O + (int64_t)item.off * D + (db < D ? db : n0);
            Tile<NT, true> t;
            tile_init(t, As, Bs, rows);
            tile_run<false, false, true>(t, n, 1, [&](int, int kb, float4* r) { load_mc<2>(W, a.ld_s, n, kb, tid / 16, 16, r); },
                                         [&](int kb, float4* r) { mask_mc<2>(n, kb, tid / 16, 16, r); },
                                         [&](int, int kb, float4* r) { load_mc<4>(O, D, n, kb, tid / 32, 8, r); },
                                         [&](int kb, float4* r) { mask_mc<4>(n, kb, tid / 32, 8, r); });
            const int64_t base = ((int64_t)slot * a.k + j0) * D + n0 + (n0 + l16 < D ? l16 : 0);
            float p[NT][4];  // all of P asked for before the first store
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                const int d = n0 + 16 * ct + l16 < D ? 16 * ct : 0;
#pragma unroll
                for (int v = 0; v < 4; ++v) p[ct][v] = a.P[base + (int64_t)min(t.row(v), rows - 1) * D + d];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double w = t.a_sum_of(v);
#pragma unroll
                for (int ct = 0; ct < NT; ++ct) {
                    if (n0 + 16 * ct + l16 < D && t.row(v) < rows)
                        a.V[base + (int64_t)t.row(v) * D + 16 * ct] = (float)(2. * (t.acc[ct][v] - w * p[ct][v]));
                }
            }
        }
        return;
    }
    const int cols = (D + DN - 1) / DN, n0 = block % cols * DN;
    TransrBlock blk;
    if (!pblock_of(a, block / cols, c, blk) || blk.all <= DP_FEW) return;
    const int db = n0 + 4 * (tid % 32), n = blk.n;
    const float* P = a.P + (int64_t)blk.slot * a.k * D + (db < D ? db : n0);
    const float* W[2];
#pragma unroll
    for (int it = 0; it < 2; ++it) W[it] = a.S + (int64_t)(blk.off + min(tid / 8 + 32 * it, n - 1)) * a.ld_s;
    Tile<NT, true> t;
    tile_init(t, As, Bs, n);
    tile_run<true, false, true>(t, a.k, 1, [&](int, int kb, float4* r) { load_kc<2>(W, a.k, kb, r); },
        [&](int kb, float4* r) {
            const int left = a.k - BK * kb - 4 * (tid % 8);  // (a row of W holds a multiple of four)
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                r[it].x = left <= 0 ? 0.f : r[it].x; r[it].y = left <= 1 ? 0.f : r[it].y;
                r[it].z = left <= 2 ? 0.f : r[it].z; r[it].w = left <= 3 ? 0.f : r[it].w;
            }
        },
        [&](int, int kb, float4* r) { load_mc<4>(P, D, a.k, kb, tid / 32, 8, r); },
        [&](int kb, float4* r) { mask_mc<4>(a.k, kb, tid / 32, 8, r); });
    if (!t.active) return;
    const float sigma = step_view(a.ids).side == KGE_NEG_HEAD ? -1.f : 1.f;
    float o[4][NT], p[4][NT];  // all of them asked for before the first store
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int64_t at = (int64_t)(blk.off + min(t.row(v), n - 1)) * D + n0 + (n0 + l16 < D ? l16 : 0);
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int d = n0 + 16 * ct + l16 < D ? 16 * ct : 0;
            o[v][ct] = a.O[at + d];
            p[v][ct] = a.PP[at + d];
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double w = t.a_sum_of(v);
        const int m = blk.off + t.row(v);
        if (t.row(v) >= n) continue;
        const int64_t at = (int64_t)m * D + n0 + l16, at_r = (int64_t)a.q.members[m] * D + n0 + l16;
        const float cp2 = 2.f * a.cpos[m];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            if (n0 + 16 * ct + l16 < D) {
                const float gp = cp2 * (o[v][ct] - p[v][ct]);  // df+/do = -2 (o - p)
                const float go = (float)(2. * (t.acc[ct][v] - w * o[v][ct])) - gp;
                a.GO[at + 16 * ct] = go;
                a.PP[at + 16 * ct] = gp;
                a.Gr[at_r + 16 * ct] = sigma * go;
            }
        }
    }
}

// what dp_few left in parts: thread per 16 bytes of a positive's row
__global__ __launch_bounds__(RT) void k_transr_go(TransrArgs a) {
    const int lanes = a.D / 4, e = blockIdx.x * RT + threadIdx.x, m = e / lanes;
    if (m >= a.b) return;
    const int64_t at = (int64_t)m * a.D + 4 * (e % lanes);
    const int i = a.q.members[m], all = a.q.count[m];
    const float cp2 = 2.f * a.cpos[m];
    const float4 o = ld4(a.O + at), p = ld4(a.PP + at);
    if (all > DP_FEW && !a.units) return;
    const int rows = a.units ? 16 : BM, parts = (a.k + rows - 1) / rows;
    double sx = 0, sy = 0, sz = 0, sw = 0;  // (in 64 bits: up to 64 parts and more, one after the other)
    for (int q0 = 0; q0 < parts; q0 += 8) {
        float4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = ld4(a.GOp + at + (q0 + q < parts ? q0 + q : 0) * (int64_t)a.b * a.D);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q0 + q < parts) { sx += v[q].x; sy += v[q].y; sz += v[q].z; sw += v[q].w; }
        }
    }
    const float4 s = make_float4((float)sx, (float)sy, (float)sz, (float)sw);
    const float4 gp = make_float4(cp2 * (o.x - p.x), cp2 * (o.y - p.y), cp2 * (o.z - p.z), cp2 * (o.w - p.w));  // df+/do = -2 (o - p)
    const float4 go = make_float4(s.x - gp.x, s.y - gp.y, s.z - gp.z, s.w - gp.w);
    st4(a.GO + at, go);
    st4(a.PP + at, gp);
    const float sigma = step_view(a.ids).side == KGE_NEG_HEAD ? -1.f : 1.f;
    st4(a.Gr + (int64_t)i * a.D + 4 * (e % lanes), make_float4(sigma * go.x, sigma * go.y, sigma * go.z, sigma * go.w));
}

// dL/do and dL/dp of a block of an item's positives (rows 2 m, 2 m + 1) times M, 128 columns, straight into their gradient rows
template <int NT>
__device__ __forceinline__ void back_positives_f32(const TransrArgs& a, int x, float* As, float* Bs) {
    const int D = a.D, tid = threadIdx.x, cols = (D + BN - 1) / BN, l16 = tid & 15;
    const int n0 = x % cols * BN, col = n0 + 4 * (tid % 32), colc = col < D ? col : n0;
    Tile<NT> t;
    int c;
    TransrBlock blk;
    if (!pblock_of(a, x / cols, c, blk)) return;
    const int n = blk.n;
    const float* M = a.R + (int64_t)blk.rel * a.rel_dim + D + colc;
    const bool head = step_view(a.ids).side == KGE_NEG_HEAD;
    tile_init(t, As, Bs, 2 * n);
    const float* pa[2];
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int row = min(tid / 8 + 32 * it, 2 * n - 1);
        pa[it] = ((row & 1) ? a.PP : a.GO) + (int64_t)(blk.off + row / 2) * D;
    }
    int i[2];  // rows 2 h, 2 h + 1 of the lane's four
#pragma unroll
    for (int h = 0; h < 2; ++h) i[h] = a.q.members[blk.off + min(t.row(2 * h) / 2, n - 1)];
    tile_run<true, false, false>(t, D, 1, [&](int, int kb, float4* r) { load_kc<2>(pa, D, kb, r); },
                                 [&](int kb, float4* r) { mask_kc<2>(D, kb, r); },
                                 [&](int, int kb, float4* r) { load_mc<4>(M, D, D, kb, tid / 32, 8, r); },
                                 [&](int kb, float4* r) { mask_mc<4>(D, kb, tid / 32, 8, r); });
    if (!t.active) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (t.row(v) >= 2 * n) continue;
        // key positions: heads 0 .. b-1, tails b .. 2b-1; even rows belong to the kept entity
        const bool to_head = head == (bool)(v & 1);
        float* out = a.Gent + ((int64_t)(to_head ? 0 : a.b) + i[v / 2]) * D;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int d = n0 + 16 * ct + l16;
            if (d < D) out[d] = t.acc[ct][v];
        }
    }
}

// V_t M_t.  The first workgroups: 64 corrupting rows of a chunk x 128 columns x a range of the chunk's items; the others: the positives.
template <int NT>
__global__ __launch_bounds__(RT, 4) void k_transr_back_f32(TransrArgs a, int neg_blocks) {
    __shared__ __attribute__((aligned(16))) float As[A_FLOATS], Bs[B_FLOATS];
    const int D = a.D, tid = threadIdx.x, cols = (D + BN - 1) / BN, l16 = tid & 15;
    Tile<NT> t;
    const bool neg = (int)blockIdx.x < neg_blocks;
    const int x = neg ? blockIdx.x : blockIdx.x - neg_blocks;
    const int n0 = x % cols * BN, col = n0 + 4 * (tid % 32), colc = col < D ? col : n0;  // D is a multiple of 4
    if (neg) {
        const int tiles = (a.k + BM - 1) / BM, seg = x / cols % a.segments, y = x / cols / a.segments;
        const int tile = y % tiles, c = y / tiles, j0 = tile * BM, rows = min(BM, a.k - j0);
        const int items = a.q.n_items[c], s0 = (int)((int64_t)items * seg / a.segments), s1 = (int)((int64_t)items * (seg + 1) / a.segments);
        tile_init(t, As, Bs, rows);
        const float* V[2];
#pragma unroll
        for (int it = 0; it < 2; ++it) V[it] = a.V + (((int64_t)c * a.g + s0) * a.k + j0 + min(tid / 8 + 32 * it, rows - 1)) * D;
        // the matrix of the item at hand and of the next one (its relation id is asked for an item ahead)
        const TransrItem* item = a.q.items + c * a.g + s0;
        const int last = s1 - s0 - 1;
        int cur = 0;
        const float* here = a.R + D + (last >= 0 ? item[0].rel : 0) * a.rel_dim + colc;
        uint32_t next = last >= 0 ? item[last > 0].rel : 0;
        tile_run<true, false, false>(t, D, s1 - s0,
            [&](int run, int kb, float4* r) {
                const float* p[2] = {V[0] + (int64_t)run * a.k * D, V[1] + (int64_t)run * a.k * D};
                load_kc<2>(p, D, kb, r);
            },
            [&](int kb, float4* r) { mask_kc<2>(D, kb, r); },
            [&](int run, int kb, float4* r) {
                if (run != cur) {
                    cur = run;
                    here = a.R + D + next * a.rel_dim + colc;
                    next = item[min(run + 1, last)].rel;
                }
                load_mc<4>(here, D, D, kb, tid / 32, 8, r);
            },
            [&](int kb, float4* r) { mask_mc<4>(D, kb, tid / 32, 8, r); });
        float* out = a.back_part + (((int64_t)seg * (a.b / a.g) + c) * a.k + j0) * D;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int d = n0 + 16 * ct + l16;
            if (d < D) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (t.row(v) < rows) out[(int64_t)t.row(v) * D + d] = t.acc[ct][v];
                }
            }
        }
        return;
    }
    back_positives_f32<NT>(a, x, As, Bs);
}

// 64 rows x 128 columns of dL/dM of an item.  K: the chunk's corrupting rows, then two rows per positive.
template <int NT>
__device__ __forceinline__ void mgrad_f32(const TransrArgs& a, int block, float* As, float* Bs) {
    const int D = a.D, tid = threadIdx.x, cols = (D + BN - 1) / BN, tiles = (D + BM - 1) / BM * cols;
    int c, slot, tile;
    TransrItem item;
    const int unit = unit_of_block(block, tiles, tile);
    if (a.units ? !unit_item_of(a, unit, c, slot, item) : !item_of(a, unit, c, slot, item)) return;
    const int n0 = tile % cols * BN, e0 = tile / cols * BM, n2 = 2 * item.n;
    const int ca = e0 + 4 * (tid % 16), cb = n0 + 4 * (tid % 32), ka = tid / 16, kb0 = tid / 32;
    const int cac = ca < D ? ca : e0, cbc = cb < D ? cb : n0;
    const float* V = a.V + (int64_t)slot * a.k * D + cac;
    const float* N = a.N + (int64_t)c * a.k * D + cbc;
    const uint32_t* ent = a.q.ent + 2 * item.off;
    uint32_t id[4];  // of the first block of positives: there when the corrupting rows are done
#pragma unroll
    for (int it = 0; it < 4; ++it) id[it] = ent[min(kb0 + 8 * it, n2 - 1)];
    Tile<NT> t;
    tile_init(t, As, Bs, min(BM, D - e0));
    tile_run<false, false, false>(t, a.k, 1, [&](int, int kb, float4* r) { load_mc<2>(V, D, a.k, kb, ka, 16, r); },
                                  [&](int kb, float4* r) { mask_mc<2>(a.k, kb, ka, 16, r); },
                                  [&](int, int kb, float4* r) { load_mc<4>(N, D, a.k, kb, kb0, 8, r); },
                                  [&](int kb, float4* r) { mask_mc<4>(a.k, kb, kb0, 8, r); });
    tile_run<false, false, false>(t, n2, 1,
        [&](int, int kb, float4* r) {
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int kk = min(BK * kb + ka + 16 * it, n2 - 1);
                r[it] = ld4(((kk & 1) ? a.PP : a.GO) + (int64_t)(item.off + kk / 2) * D + cac);
            }
        },
        [&](int kb, float4* r) { mask_mc<2>(n2, kb, ka, 16, r); },
        [&](int, int kb, float4* r) {
            if (kb > 0) {
#pragma unroll
                for (int it = 0; it < 4; ++it) id[it] = ent[min(BK * kb + kb0 + 8 * it, n2 - 1)];
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) r[it] = ld4(a.E + (int64_t)id[it] * D + cbc);
        },
        [&](int kb, float4* r) { mask_mc<4>(n2, kb, kb0, 8, r); });
    float* out = a.GM + (int64_t)slot * D * D;
    const int l16 = tid & 15;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int e = e0 + t.row(v);
        if (e >= D) continue;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int d = n0 + 16 * ct + l16;
            if (d < D) out[(int64_t)e * D + d] = t.acc[ct][v];
        }
    }
}

// The first workgroups: matrix gradients; the others, where k_transr_project_units has done the corrupting rows: back_positives.
template <int NT>
__global__ __launch_bounds__(RT, 4) void k_transr_mgrad_f32(TransrArgs a, int blocks, int back) {
    __shared__ __attribute__((aligned(16))) float As[A_FLOATS], Bs[B_FLOATS];
    const int block = flat_block();
    if (block < blocks) mgrad_f32<NT>(a, block, As, Bs);
    else if (block - blocks < back) back_positives_f32<NT>(a, block - blocks, As, Bs);
}

// The same on the bf16 matrix cores.
template <int NT>
__device__ __forceinline__ void back_positives(const TransrArgs& a, int x, uint16_t* Bs) {
    const int D = a.D, tid = threadIdx.x, cols = (D + BN - 1) / BN, l16 = tid & 15;
    const int n0 = x % cols * BN, col = n0 + 4 * (tid % 32), colc = col < D ? col : n0;
    SplitTile<NT> t;
    int c;
    TransrBlock blk;
    if (!pblock_of(a, x / cols, c, blk)) return;
    const int n = blk.n;
    const float* M = a.R + (int64_t)blk.rel * a.rel_dim + D + colc;
    const bool head = step_view(a.ids).side == KGE_NEG_HEAD;
    split_init(t, 2 * n);
    const int row = min(t.a_row(), 2 * n - 1);
    const float* pa = ((row & 1) ? a.PP : a.GO) + (int64_t)(blk.off + row / 2) * D;
    int i[2];  // rows 2 h, 2 h + 1 of the lane's four
#pragma unroll
    for (int h = 0; h < 2; ++h) i[h] = a.q.members[blk.off + min(t.row(2 * h) / 2, n - 1)];
    split_run(t, Bs, D, 1, [&](int, int kb, float4 (&r)[2]) { load_row(pa, BK * kb + t.a_k(), D, r); },
                     [&](int kb, float4 (&r)[2]) { mask_row(BK * kb + t.a_k(), D, r); },
                     [&](int, int kb, float4* r) { load_mc<4>(M, D, D, kb, 4 * (tid / 32), 1, r); },
                     [&](int kb, float4* r) { mask_mc<4>(D, kb, 4 * (tid / 32), 1, r); });
    split_sum(t);
    if (!t.active) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (t.row(v) >= 2 * n) continue;
        // key positions: heads 0 .. b-1, tails b .. 2b-1; even rows belong to the kept entity
        const bool to_head = head == (bool)(v & 1);
        float* out = a.Gent + ((int64_t)(to_head ? 0 : a.b) + i[v / 2]) * D;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int d = n0 + 16 * ct + l16;
            if (d < D) out[d] = t.acc[ct][v];
        }
    }
}

template <int NT>
__global__ __launch_bounds__(RT, 3) void k_transr_back(TransrArgs a, int neg_blocks) {
    __shared__ __attribute__((aligned(16))) uint16_t Bs[3 * 16 * NT * SP];
    const int D = a.D, tid = threadIdx.x, cols = (D + BN - 1) / BN, l16 = tid & 15;
    SplitTile<NT> t;
    const bool neg = (int)blockIdx.x < neg_blocks;
    const int x = neg ? blockIdx.x : blockIdx.x - neg_blocks;
    const int n0 = x % cols * BN, col = n0 + 4 * (tid % 32), colc = col < D ? col : n0;  // D is a multiple of 4
    if (neg) {
        const int tiles = (a.k + BM - 1) / BM, seg = x / cols % a.segments, y = x / cols / a.segments;
        const int tile = y % tiles, c = y / tiles, j0 = tile * BM, rows = min(BM, a.k - j0);
        const int items = a.q.n_items[c], s0 = (int)((int64_t)items * seg / a.segments), s1 = (int)((int64_t)items * (seg + 1) / a.segments);
        split_init(t, rows);
        const float* V = a.V + (((int64_t)c * a.g + s0) * a.k + j0 + min(t.a_row(), rows - 1)) * D;
        // the matrix of the item at hand and of the next one (its relation id is asked for an item ahead)
        const TransrItem* item = a.q.items + c * a.g + s0;
        const int last = s1 - s0 - 1;
        int cur = 0;
        const float* here = a.R + D + (last >= 0 ? item[0].rel : 0) * a.rel_dim + colc;
        uint32_t next = last >= 0 ? item[last > 0].rel : 0;
        split_run(t, Bs, D, s1 - s0,
            [&](int run, int kb, float4 (&r)[2]) { load_row(V + (int64_t)run * a.k * D, BK * kb + t.a_k(), D, r); },
            [&](int kb, float4 (&r)[2]) { mask_row(BK * kb + t.a_k(), D, r); },
            [&](int run, int kb, float4* r) {
                if (run != cur) {
                    cur = run;
                    here = a.R + D + next * a.rel_dim + colc;
                    next = item[min(run + 1, last)].rel;
                }
                load_mc<4>(here, D, D, kb, 4 * (tid / 32), 1, r);
            },
            [&](int kb, float4* r) { mask_mc<4>(D, kb, 4 * (tid / 32), 1, r); });
        split_sum(t);
        float* out = a.back_part + (((int64_t)seg * (a.b / a.g) + c) * a.k + j0) * D;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int d = n0 + 16 * ct + l16;
            if (d < D) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (t.row(v) < rows) out[(int64_t)t.row(v) * D + d] = t.acc[ct][v];
                }
            }
        }
        return;
    }
    back_positives<NT>(a, x, Bs);
}

template <int NT>
__device__ __forceinline__ void mgrad(const TransrArgs& a, int block, uint16_t* Bs) {
    const int D = a.D, tid = threadIdx.x, cols = (D + BN - 1) / BN, tiles = (D + BM - 1) / BM * cols;
    int c, slot, tile;
    TransrItem item;
    const int unit = unit_of_block(block, tiles, tile);
    if (a.units ? !unit_item_of(a, unit, c, slot, item) : !item_of(a, unit, c, slot, item)) return;
    const int n0 = tile % cols * BN, e0 = tile / cols * BM, n2 = 2 * item.n;
    const int cb = n0 + 4 * (tid % 32), kb0 = 4 * (tid / 32), cbc = cb < D ? cb : n0;
    SplitTile<NT> t;
    split_init(t, min(BM, D - e0));
    const int e = min(e0 + t.a_row(), D - 1);
    const float* V = a.V + (int64_t)slot * a.k * D + e;
    const float* N = a.N + (int64_t)c * a.k * D + cbc;
    const uint32_t* ent = a.q.ent + 2 * item.off;
    uint32_t id[4];  // of the first block of positives: there when the corrupting rows are done
#pragma unroll
    for (int it = 0; it < 4; ++it) id[it] = ent[min(kb0 + it, n2 - 1)];
    // A is stored with K along its rows: a lane's eight values are eight rows of 16 consecutive lanes' floats
    auto eight = [&](float4 (&r)[2], auto at) {
        r[0] = make_float4(at(0), at(1), at(2), at(3));
        r[1] = make_float4(at(4), at(5), at(6), at(7));
    };
    auto mask_eight = [&](int k, int K, float4 (&r)[2]) {
        r[0] = make_float4(k < K ? r[0].x : 0.f, k + 1 < K ? r[0].y : 0.f, k + 2 < K ? r[0].z : 0.f, k + 3 < K ? r[0].w : 0.f);
        r[1] = make_float4(k + 4 < K ? r[1].x : 0.f, k + 5 < K ? r[1].y : 0.f, k + 6 < K ? r[1].z : 0.f, k + 7 < K ? r[1].w : 0.f);
    };
    split_run(t, Bs, a.k, 1,
        [&](int, int kb, float4 (&r)[2]) {
            const int k = BK * kb + t.a_k();
            eight(r, [&](int j) { return V[(int64_t)min(k + j, a.k - 1) * D]; });
        },
        [&](int kb, float4 (&r)[2]) { mask_eight(BK * kb + t.a_k(), a.k, r); },
        [&](int, int kb, float4* r) { load_mc<4>(N, D, a.k, kb, kb0, 1, r); },
        [&](int kb, float4* r) { mask_mc<4>(a.k, kb, kb0, 1, r); });
    split_run(t, Bs, n2, 1,
        [&](int, int kb, float4 (&r)[2]) {
            const int k = BK * kb + t.a_k();
            eight(r, [&](int j) {
                const int kk = min(k + j, n2 - 1);
                return ((kk & 1) ? a.PP : a.GO)[(int64_t)(item.off + kk / 2) * D + e];
            });
        },
        [&](int kb, float4 (&r)[2]) { mask_eight(BK * kb + t.a_k(), n2, r); },
        [&](int, int kb, float4* r) {
            if (kb > 0) {
#pragma unroll
                for (int it = 0; it < 4; ++it) id[it] = ent[min(BK * kb + kb0 + it, n2 - 1)];
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) r[it] = ld4(a.E + (int64_t)id[it] * D + cbc);
        },
        [&](int kb, float4* r) { mask_mc<4>(n2, kb, kb0, 1, r); });
    split_sum(t);
    float* out = a.GM + (int64_t)slot * D * D;
    const int l16 = tid & 15;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int er = e0 + t.row(v);
        if (er >= D) continue;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int d = n0 + 16 * ct + l16;
            if (d < D) out[(int64_t)er * D + d] = t.acc[ct][v];
        }
    }
}

template <int NT>
__global__ __launch_bounds__(RT, 3) void k_transr_mgrad(TransrArgs a, int blocks, int back) {
    __shared__ __attribute__((aligned(16))) uint16_t Bs[3 * 16 * NT * SP];
    const int block = flat_block();
    if (block < blocks) mgrad<NT>(a, block, Bs);
    else if (block - blocks < back) back_positives<NT>(a, block - blocks, Bs);
}

struct TransrUpdArgs {
    float* T;             // relation table [n_rel x (D + D*D)]
    float* St;            // its Adagrad accumulator
    const uint32_t* key;  // sorted relation ids of the step
    const uint32_t* pos;  // position in the mini-batch of each sorted entry
    const int* slot_of;   // item (unit) slot of the positives that are the first of theirs, else -1
    int n, D, rows_per_slab, slabs;
    int64_t rel_dim;
    const float* Gr;
    const float* GM;
    float lr, eps;
    PartialRows rest;     // gradient rows of the corrupting entities, still in parts
    int share, rest_blocks;
};

// Workgroup (p, slab): slab 0 is the translation, slab s > 0 rows (s - 1) * rows_per_slab .. of the matrix.  If sorted
// position p is the last of its run of equal relation ids, the workgroup sums the run's gradient rows for its slab in
// sorted order (translation: a row per positive; matrix: one per item) and applies Adagrad.
__global__ __launch_bounds__(RT) void k_transr_update(TransrUpdArgs a) {
    const int tid = threadIdx.x, block = flat_block(), rows_blocks = a.n * a.slabs;
    if (block >= rows_blocks) {
        if (block < rows_blocks + a.rest_blocks) sum_partial_rows<RT>(a.rest, a.share, block - rows_blocks, a.rest_blocks);
        return;
    }
    const int p = block / a.slabs, slab = block % a.slabs;
    const uint32_t key = a.key[p];
    if (p + 1 < a.n && a.key[p + 1] == key) return;  // the run goes on (same decision in every thread)
    __shared__ int first_other, n_rows;
    __shared__ int lrow[RT];
    const int D = a.D;
    const int width = slab == 0 ? D : a.rows_per_slab * D, lanes = width / 4;
    const int groups = RT / lanes, grp = tid / lanes;  // thread groups share out the rows of the run; the first applies the sum
    const bool act = grp < groups;
    const int e = act ? 4 * (tid - grp * lanes) : 0;
    const int64_t in_row = slab == 0 ? e : (int64_t)D + (int64_t)(slab - 1) * a.rows_per_slab * D + e;
    const int64_t off = (int64_t)key * a.rel_dim + in_row;
    const float* G = slab == 0 ? a.Gr + e : a.GM + (int64_t)(slab - 1) * a.rows_per_slab * D + e;
    const int64_t g_stride = slab == 0 ? D : (int64_t)D * D;
    float4 x = f4(0.f), s = f4(0.f);
    if (grp == 0) { x = ld4(a.T + off); s = ld4(a.St + off); }
    if (tid == 0) first_other = 1 << 30;
    __syncthreads();
    for (int base = 1;; base += RT) {
        const int q = p - (base + tid);
        const bool differs = q < 0 || a.key[q < 0 ? 0 : q] != key;
        const unsigned long long bal = __ballot(differs);
        if ((tid & 63) == 0 && bal) atomicMin(&first_other, base + tid + __builtin_ctzll(bal));
        __syncthreads();
        const bool found = first_other < (1 << 30);
        __syncthreads();
        if (found) break;
    }
    const int start = p - first_other + 1;
    float4 g = f4(0.f);
    __shared__ __attribute__((aligned(16))) float4 part[RT];
    __shared__ int wcount[RT / 64];
    for (int c0 = start; c0 <= p; c0 += RT) {
        // the rows of this part of the run, in order
        int row = -1;
        if (c0 + tid <= p) {
            row = (int)a.pos[c0 + tid];
            if (slab > 0) row = a.slot_of[row];
        }
        const unsigned long long bal = __ballot(row >= 0);
        __syncthreads();
        if ((tid & 63) == 0) wcount[tid >> 6] = __popcll(bal);
        __syncthreads();
        int at = __popcll(bal & ((1ull << (tid & 63)) - 1));
        for (int w = 0; w < tid >> 6; ++w) at += wcount[w];
        if (row >= 0) lrow[at] = row;
        if (tid == 0) { n_rows = 0; for (int w = 0; w < RT / 64; ++w) n_rows += wcount[w]; }
        __syncthreads();
        const int m = n_rows;
        if (act) {
#pragma unroll 4
            for (int j = grp; j < m; j += groups) {
                const float4 t = ld4(G + (int64_t)lrow[j] * g_stride);
                g.x += t.x; g.y += t.y; g.z += t.z; g.w += t.w;
            }
        }
    }
    if (groups > 1) {
        part[tid] = g;
        __syncthreads();
        for (int g2 = 1; grp == 0 && g2 < groups; ++g2) {
            const float4 t = part[g2 * lanes + tid];
            g.x += t.x; g.y += t.y; g.z += t.z; g.w += t.w;
        }
    }
    if (grp == 0) {
        adagrad4(g, x, s, a.lr, a.eps);
        st4(a.St + off, s);
        st4(a.T + off, x);
    }
}

TransrArgs make_args(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, int gsz, float gamma) {
    TransrArgs a;
    const int D = c->cfg.ent_dim;
    a.E = E; a.R = R; a.ids = ids; a.b = ids.b; a.D = D; a.k = k; a.g = gsz; a.ld_s = c->ld_s;
    a.n_ent = c->cfg.num_entities; a.n_rel = c->cfg.num_relations; a.rel_dim = c->cfg.rel_dim;
    a.max_items = transr_max_items(gsz, a.n_rel);
    a.max_pblocks = transr_max_pblocks(gsz, a.n_rel);
    a.gamma = gamma; a.wk = 1.f / ((float)(k > 0 ? k : 1) * (float)ids.b);
    a.out_w = 0; a.train = 1; a.segments = 1; a.units = 0; a.unit_rows = UROWS;
    a.q = c->tr_groups;
    a.O = c->O; a.PP = c->PP; a.P = c->P3; a.V = c->P3 + kge_transr_p_floats(c->cfg);
    a.N = c->Nst; a.S = c->S; a.GO = c->GO; a.GOp = c->tr_go_part;
    a.fpos = c->fpos; a.pos_out = nullptr; a.cpos = c->cpos; a.row_loss = c->row_loss; a.loss_part = c->neg_loss_part;
    a.Gent = c->Gent; a.Gr = c->Grel; a.GM = c->Grel + (int64_t)c->cfg.max_batch * D;
    a.back_part = c->tr_back_part;
    return a;
}

// Ranges of a chunk's items in the back-projection: about three workgroups per CU, at least one item each.
int back_segments(const TransrArgs& a) {
    const int base = (a.b / a.g) * ((a.k + BM - 1) / BM) * ((a.D + BN - 1) / BN);
    int s = (KGE_TRANSR_BACK_WGS + base - 1) / base;
    return s > a.max_items ? a.max_items : s;
}

// Everything between phi and the matrix gradients in k_transr_project_units?  Wherever it can be.  us per step, launches of their own ->
// units (b, g, k, D, relations)  1024, 128, 256, 100, 1345 244 -> 190;  D 128 280 -> 220;  D 64 150 -> 111;  k 500, D 32 148 -> 120;  20 relations
// 145 -> 130;  1024, 256, 640, 100, 1345 491 -> 330;  1024, 1024, 16, 100, 20 137 -> 102;  2000, 16, 8, 128, 1345 255 -> 253.  The only shapes found
// where launches of their own are faster have rows of more than 96 floats, few corrupting rows, chunks of up to 128 and some ten positives
// per relation and chunk, whose units a single wave per SIMD works through: 1024, 128, 8, 128, 5 98.6 -> 102.5;  16, 128, 10 95.8 -> 98.6;  32, 128, 20
// 98.6 -> 101.0;  16, 100, 20 89.5 -> 90.5;  64, 100, 20 97.2 -> 96.2;  512, 64, 16, 128, 4 84.8 -> 88.7, k 40 99.9 -> 92.9.
bool may_take_units(const kge_config& cfg) { return cfg.adv_temperature == 0.f && cfg.loss == KGE_LOSS_LOGISTIC && cfg.ent_dim <= BN; }
bool in_units(const kge_ctx* c, bool form_w) { return form_w && may_take_units(c->cfg); }
// Corrupting rows per workgroup: 128, two waves per SIMD, which is what fills the chip; 64, one wave per SIMD, where the units are so few that
// half as many rows still leave no workgroup to a second round.  (us per step, 128 -> 64: 1024, 1024, 72, 128, 5 132 -> 119;  1024, 128, 100, 128, 5 127 ->
// 114, launches of their own 111;  256, 256, 256, 64, 20 71.6 -> 67.3;  32 and 16 rows: no change.)
int unit_rows(const TransrArgs& a) {
    return (int64_t)(a.b / a.g) * a.max_pblocks * ((a.k + UROWS / 2 - 1) / (UROWS / 2)) <= KGE_TRANSR_UNIT_WGS ? UROWS / 2 : UROWS;
}
// Ranges of a chunk's units.  A workgroup has a CU to itself (rows of up to 32 floats: half of one), so a grid of a few workgroups
// more than the chip holds takes twice the time: of the numbers that fill one to eight rounds, the one whose rounds times (units of a
// range, and one for its start and its gradient rows) is least.  Units per chunk are known on the device only; two thirds of the most
// there can be is what a Zipf-distributed graph has.  us per step, ceil(256 / workgroups per range) -> this (b, g, k, D, relations): 1024,
// 256, 640, 100, 1345 425 -> 330 (260 workgroups -> 240);  1024, 128, 300, 100 274 -> 238;  1000, 200, 700, 100 472 -> 370;  1040, 16, 256, 100
// 333 -> 301 (260 -> 390);  1600, 50, 640, 32 241 -> 215;  1000, 1000, 200, 32 78.1 -> 81.3 (256 -> 512).
int unit_segments(const TransrArgs& a) {
    const int64_t chunks = a.b / a.g, base = chunks * ((a.k + a.unit_rows - 1) / a.unit_rows), slots = a.D <= 32 ? 2 * KGE_TRANSR_UNIT_WGS : KGE_TRANSR_UNIT_WGS;
    const int64_t rows = chunks * a.k, room = (rows + (chunks + KGE_TRANSR_BACK_WGS) * BM) / rows;  // (kge_transr_back_floats)
    const int64_t most = room < a.max_pblocks ? room : a.max_pblocks;
    auto cost = [&](int64_t s) { return (double)((base * s + slots - 1) / slots) * (1. + 0.65 * a.max_pblocks / (double)s); };
    int64_t best = 1;
    for (int r = 1; r <= 8; ++r) {
        const int64_t fill = r * slots / base, s = fill < most ? fill : most;
        if (s > 1 && cost(s) < cost(best)) best = s;
    }
    return (int)best;
}

template <int NT>
auto back_kernel() {
    if constexpr (NT < SPLIT_FROM) return k_transr_back_f32<NT>;
    else return k_transr_back<NT>;
}
template <int NT>
auto mgrad_kernel() {
    if constexpr (NT < SPLIT_FROM) return k_transr_mgrad_f32<NT>;
    else return k_transr_mgrad<NT>;
}

// column tiles of 16 per workgroup
#define KGE_BY_COLUMNS(D, LAUNCH)                                                                     \
    do {                                                                                              \
        switch (((D) < BN ? (D) + 15 : BN) / 16) {                                                    \
        case 1: case 2: LAUNCH(2); break;                                                             \
        case 3: LAUNCH(3); break;                                                                     \
        case 4: LAUNCH(4); break;                                                                     \
        case 5: LAUNCH(5); break;                                                                     \
        case 6: LAUNCH(6); break;                                                                     \
        case 7: LAUNCH(7); break;                                                                     \
        default: LAUNCH(8); break;                                                                    \
        }                                                                                             \
    } while (0)

}  // namespace

// train: what later launches read stays in the order of the items' positives; otherwise the outputs are the caller's
void kge_transr_phi(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int gsz, float gamma, float* pos_out, bool train,
                    bool form_w, hipStream_t st) {
    TransrArgs a = make_args(c, E, R, ids, 0, gsz, gamma);
    a.pos_out = pos_out; a.train = train; a.units = train && in_units(c, form_w);
#define L(NT) KGE_LAUNCH(c, k_transr_phi<NT>, dim3(ids.b / gsz * a.max_pblocks), dim3(RT), 0, st, a)
    KGE_BY_COLUMNS(a.D, L);
#undef L
}

int kge_transr_project(kge_ctx* c, const float* R, const StepIds& ids, int k, int gsz, float gamma, float* out, int ld_out, bool train,
                       bool form_w, hipStream_t st) {
    TransrArgs a = make_args(c, nullptr, R, ids, k, gsz, gamma);
    if (train && in_units(c, form_w)) {
        const int chunks = ids.b / gsz;
        float* rows = a.Gent + (int64_t)2 * ids.b * a.D;
        const int64_t stride = (int64_t)chunks * k * a.D;
        a.unit_rows = unit_rows(a);
        a.segments = unit_segments(a);
        c->neg_partial = {c->tr_back_part, rows, a.segments, stride, stride / 4};
        if (a.segments == 1) a.back_part = rows;
        const int wgs = chunks * ((k + a.unit_rows - 1) / a.unit_rows) * a.segments;
#define L(NT) KGE_LAUNCH(c, k_transr_project_units<NT>, dim3(wgs), dim3(UT), 0, st, a)
        KGE_BY_COLUMNS(a.D, L);
#undef L
        return wgs;
    }
    a.S = out; a.ld_s = ld_out; a.out_w = form_w; a.train = train;
    const int blocks = pblock_blocks(a, (k + BM - 1) / BM);
#define L(NT) KGE_LAUNCH(c, k_transr_project<NT>, flat_grid(blocks), dim3(RT), 0, st, a, blocks)
    KGE_BY_COLUMNS(a.D, L);
#undef L
    return form_w ? blocks : 0;
}

void kge_transr_dp(kge_ctx* c, const StepIds& ids, int k, int gsz, bool form_w, hipStream_t st) {
    TransrArgs a = make_args(c, nullptr, nullptr, ids, k, gsz, 0.f);
    a.units = in_units(c, form_w);
    if (a.units) {
        KGE_LAUNCH(c, k_transr_go, dim3((ids.b * (a.D / 4) + RT - 1) / RT), dim3(RT), 0, st, a);
        return;
    }
    const int cols = (a.D + DN - 1) / DN, go_blocks = (ids.b / gsz * a.max_pblocks * cols + 7) / 8 * 8;
    const int blocks = go_blocks + item_blocks(a, (k + BM - 1) / BM);
    const dim3 grid = flat_grid(blocks);
    if (a.D <= 32) KGE_LAUNCH(c, k_transr_dp<2>, grid, dim3(RT), 0, st, a, go_blocks, blocks);
    else if (a.D <= 48) KGE_LAUNCH(c, k_transr_dp<3>, grid, dim3(RT), 0, st, a, go_blocks, blocks);
    else KGE_LAUNCH(c, k_transr_dp<4>, grid, dim3(RT), 0, st, a, go_blocks, blocks);
    hipLaunchKernelGGL(k_transr_go, dim3((ids.b * (a.D / 4) + RT - 1) / RT), dim3(RT), 0, st, a);
}

void kge_transr_back(kge_ctx* c, const float* R, const StepIds& ids, int k, int gsz, bool form_w, hipStream_t st) {
    if (in_units(c, form_w)) return;  // k_transr_project_units and k_transr_mgrad
    TransrArgs a = make_args(c, nullptr, R, ids, k, gsz, 0.f);
    const int chunks = ids.b / gsz, cols = (a.D + BN - 1) / BN;
    a.segments = back_segments(a);
    float* out = a.Gent + (int64_t)2 * ids.b * a.D;
    const int64_t stride = (int64_t)chunks * k * a.D;
    c->neg_partial = {c->tr_back_part, out, a.segments, stride, stride / 4};
    if (a.segments == 1) a.back_part = out;
    const int neg_blocks = chunks * ((k + BM - 1) / BM) * a.segments * cols;
    const dim3 grid(neg_blocks + chunks * a.max_pblocks * cols);
#define L(NT) KGE_LAUNCH(c, back_kernel<NT>(), grid, dim3(RT), 0, st, a, neg_blocks)
    KGE_BY_COLUMNS(a.D, L);
#undef L
}

void kge_transr_mgrad(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int k, int gsz, bool form_w, hipStream_t st) {
    TransrArgs a = make_args(c, E, R, ids, k, gsz, 0.f);
    a.units = in_units(c, form_w);
    const int tiles = ((a.D + BM - 1) / BM) * ((a.D + BN - 1) / BN), blocks = a.units ? pblock_blocks(a, tiles) : item_blocks(a, tiles);
    const int back = a.units ? ids.b / gsz * a.max_pblocks : 0;  // (rows of one column tile)
#define L(NT) KGE_LAUNCH(c, mgrad_kernel<NT>(), flat_grid((int64_t)blocks + back), dim3(RT), 0, st, a, blocks, back)
    KGE_BY_COLUMNS(a.D, L);
#undef L
}

void kge_transr_update(kge_ctx* c, float* R, float* SR, const StepIds& ids, float lr, bool form_w, hipStream_t st) {
    TransrUpdArgs a;
    const int D = c->cfg.ent_dim;
    int rows = 1024 / D;  // matrix rows per workgroup: the largest divisor of D that keeps a slab within 1024 floats
    while (D % rows != 0) --rows;
    a.T = R; a.St = SR; a.key = c->rkey[c->rbuf]; a.pos = c->rpos[c->rbuf]; a.slot_of = in_units(c, form_w) ? c->tr_groups.unit_of : c->tr_groups.slot_of;
    a.n = ids.b; a.D = D; a.rows_per_slab = rows; a.slabs = D / rows + 1; a.rel_dim = c->cfg.rel_dim;
    a.Gr = c->Grel; a.GM = c->Grel + (int64_t)c->cfg.max_batch * D;
    a.lr = lr; a.eps = c->eps;
    a.rest = c->neg_partial;
    a.rest_blocks = partial_rows_blocks(a.rest, a.share);
    KGE_LAUNCH(c, k_transr_update, flat_grid(ids.b * a.slabs + a.rest_blocks), dim3(RT), 0, st, a);
}

// bytes of the workspace that the items of a mini-batch take (base null: only counted)
size_t kge_transr_carve_groups(const kge_config& cfg, char* base, TransrGroups* q) {
    const size_t B = cfg.max_batch, C = cfg.max_chunks, PBS = B + B / PB + C;
    size_t off = 0;
    auto take = [&](size_t bytes) { char* p = base + off; off += (bytes + 255) / 256 * 256; return p; };
    q->items = (TransrItem*)take(B * sizeof(TransrItem)); q->pblocks = (TransrBlock*)take(PBS * sizeof(TransrBlock));
    q->first = (int*)take(B * 4); q->rank = (int*)take(B * 4); q->count = (int*)take(B * 4); q->slot_of = (int*)take(B * 4); q->unit_of = (int*)take(B * 4);
    q->members = (int*)take(B * 4); q->ent = (uint32_t*)take(2 * B * 4);
    q->n_items = (int*)take(C * 4); q->n_pblocks = (int*)take(C * 4);
    return off;
}
// floats of partial rows: of the back-projection (its workgroups write a tile each), of dL/do
size_t kge_transr_back_floats(const kge_config& cfg) {
    const size_t D = cfg.ent_dim, NR = (size_t)cfg.max_chunks * (cfg.max_neg_per_chunk > 0 ? cfg.max_neg_per_chunk : 1);
    return (NR + (size_t)cfg.max_chunks * BM + (size_t)KGE_TRANSR_BACK_WGS * BM) * D;
}
size_t kge_transr_go_floats(const kge_config& cfg) {
    const size_t K = cfg.max_neg_per_chunk, in_units = (K < KGE_SHORT_SCORES ? K : KGE_SHORT_SCORES) / 16 + 1, parts = K / BM + 1;
    return (size_t)cfg.max_batch * cfg.ent_dim * (may_take_units(cfg) && in_units > parts ? in_units : parts);
}
// and of the projections that training steps keep: none where all of them run in units
size_t kge_transr_p_floats(const kge_config& cfg) {
    return may_take_units(cfg) && cfg.max_neg_per_chunk <= KGE_SHORT_SCORES ? 0 : (size_t)cfg.max_batch * cfg.max_neg_per_chunk * cfg.ent_dim;
}
