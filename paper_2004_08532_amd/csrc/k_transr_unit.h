// TransR training steps with W formed on the way (uniform weights, logistic loss), rows of up to 128 floats: everything between the
// positives' o and p and the matrix gradients in one pass over the units, the blocks of up to 32 positives of an item.
//
// A workgroup of eight waves owns 128 corrupting rows of a chunk (64 where units are few) and a range of its units.  The rows, split into three bf16
// parts (k_split.h), stay in registers (16 rows per wave) for all of its units, and so do the gradient rows it adds up.  Per unit:
//   M in three parts to LDS;  P = N M^T, scores, W, V = sum 2 W (o - P), parts of dL/do (a row per positive and wave);
//   gradient rows += V M, with M read from LDS transposed; V goes through LDS to become the left operand
// V is stored for k_transr_mgrad; P, scores and W are not.  (Launches of their own read N, M and V again, split all of them again for
// every 64 rows, and stored P or V in between.)
// What bounds it: one workgroup per CU (90 to 150 KB of LDS and 170 to 256 registers for rows of more than 32 floats), two waves per SIMD
// whose phases hardly overlap.  FB15k-sized (D 100, 1332 units, 5.2 per workgroup, 1.5 positives per unit): 75 us; cycles per unit: M in three
// parts and o to LDS 3,100, first product 4,500 (its matrix instructions 2,700 per wave), scores and W 1,800, V and dL/do 1,900, V through LDS and
// into parts 2,300, second product 4,900, barriers 4,200, the next M asked for 800; 23,500 in all.  (D 128 26,100, D 64 9,500.)
// Tried: M stored a second time, transposed, for the second product, and the sums of both products in registers throughout (104
// spills) 152 us instead of 84; sums of four positives first 102 us.
#pragma once

namespace {

constexpr int UT = 512, UROWS = 128;  // threads, most corrupting rows per workgroup
constexpr int UVP = 68;               // pitch of the staged V: 16-byte reads of sixteen rows free of conflicts

// How a chunk's units are dealt to the workgroups: by their cost, what a unit takes but for its positives (20,000 cycles at D 100) against what
// one of these adds (2,400).
constexpr int UNIT_COST = 8, POSITIVE_COST = 1;

// LDS position (bf16 elements) of column `col` (a multiple of 4) of row `row` of a part of M: rows of 128 columns, 16-byte groups
// permuted by row so that neither sixteen rows' reads of one group (left product) nor the transposing reads of 4 x 16 blocks of
// rows 8 q .. 8 q + 3 and 8 q + 4 .. 8 q + 7 (right product) meet in a bank.
__device__ __forceinline__ int unit_at(int row, int col) {
    const int f = 2 * (row & 3) + (row & 8) + (row >> 2 & 1);
    return 128 * row + ((col & ~7) ^ (8 * f)) + (col & 4);
}

__device__ __forceinline__ void wave_fence() {  // LDS traffic of one wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Sums over the four quarters of a wave of four values; quarter q gets that of value q (vector ALU swaps, no LDS)
template <class T>
__device__ __forceinline__ T sum_quads(const T (&x)[4]) {
    struct Words { uint32_t w[sizeof(T) / 4]; };
    auto exchanged = [](T a, T b, auto swap) {  // a and b with what swap exchanges of them, added
        Words u = __builtin_bit_cast(Words, a), v = __builtin_bit_cast(Words, b);
#pragma unroll
        for (size_t i = 0; i < sizeof(T) / 4; ++i) {
            const auto r = swap(u.w[i], v.w[i]);
            u.w[i] = r[0]; v.w[i] = r[1];
        }
        return __builtin_bit_cast(T, u) + __builtin_bit_cast(T, v);
    };
    auto halves = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_permlane32_swap(a, b, false, false); };
    auto rows = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_permlane16_swap(a, b, false, false); };
    return exchanged(exchanged(x[0], x[2], halves), exchanged(x[1], x[3], halves), rows);
}

// The units of range `seg` of a chunk: cut[0] .. cut[1] - 1, for every thread behind the next barrier.  Returns the chunk's number of units.
__device__ __forceinline__ int unit_cut(const TransrArgs& a, int c, int seg, const TransrBlock* units, int* cut) {
    const int n_units = a.q.n_pblocks[c], tid = threadIdx.x;
    if (tid < 2) cut[tid] = 0;
    __syncthreads();
    const int64_t total = (int64_t)UNIT_COST * n_units + (int64_t)POSITIVE_COST * a.g;
    const int64_t lo = total * seg / a.segments, hi = total * (seg + 1) / a.segments;
    int n_lo = 0, n_hi = 0;
    for (int e = tid; e < n_units; e += UT) {
        const int64_t before = (int64_t)UNIT_COST * e + (int64_t)POSITIVE_COST * (units[e].off - c * a.g);
        n_lo += before < lo;
        n_hi += before < hi;
    }
    if (n_lo) atomicAdd(&cut[0], n_lo);
    if (n_hi) atomicAdd(&cut[1], n_hi);
    return n_units;
}

template <int NT>
__global__ __launch_bounds__(UT) void k_transr_project_units(TransrArgs a) {
    constexpr int KS = (NT + 1) / 2, W = 16 * NT, BLOCKS = (KS * KS + 7) / 8;  // K steps, columns, 32 x 32 blocks of M that a wave brings to LDS
    constexpr int PART = 32 * KS * 128;
    __shared__ __attribute__((aligned(16))) uint16_t Ms[3 * PART];
    __shared__ __attribute__((aligned(16))) float Vs[8][16 * UVP], Os[PB * W];
    __shared__ int cut[2];
    __shared__ float part[8];
    const int D = a.D, tid = threadIdx.x, w = tid >> 6, lane = tid & 63, l16 = lane & 15, quad = lane >> 4;
    const int tiles = (a.k + a.unit_rows - 1) / a.unit_rows;
    const int seg = blockIdx.x % a.segments, tile = blockIdx.x / a.segments % tiles, c = blockIdx.x / a.segments / tiles;
    const int j0 = tile * a.unit_rows, rows = min(a.unit_rows, a.k - j0);
    const bool active = 16 * w < rows;
    const TransrBlock* units = a.q.pblocks + (int64_t)c * a.max_pblocks;

    const int n_units = unit_cut(a, c, seg, units, cut);  // this workgroup's: cut[0] .. cut[1] - 1, behind the next barrier
    // the rows, in three parts
    Split8 nf[KS];
    {
        const float* N = a.N + ((int64_t)c * a.k + j0 + min(16 * w + l16, rows - 1)) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            float4 r[2];
            load_row(N, BK * ks + 8 * quad, D, r);
            mask_row(BK * ks + 8 * quad, D, r);
            if (__any(is_large(fmaxf(magnitude(r[0]), magnitude(r[1]))))) nf[ks] = split_row<true>(r[0], r[1]);
            else nf[ks] = split_row<false>(r[0], r[1]);
        }
    }
    __syncthreads();
    const int first = cut[0], end = cut[1];

    // A lane's share of M: 4 x 4 elements (rows me + i, columns md + ..) of block w + 8 q, an 8 x 8 arrangement of lanes
    struct Share { float4 m[BLOCKS][4]; };
    // The addresses of M's parts are formed from lx; where rows have more than 64 floats, again for every unit and product: some forty of
    // them, kept throughout, left the products too few registers (D 128: 47 spills -> 2, FB15k-sized 242 -> 221 us per step; D 100: 10 -> 0, no
    // change).  Shorter rows have the registers (D 64: 112.1 us, formed again 114.7).
    int lx = lane;
    auto again = [&]() { if (NT > 4) asm volatile("" : "+v"(lx)); };
    auto me = [&](int q) { return (w + 8 * q) / KS * 32 + 4 * (lx >> 3); };
    auto md = [&](int q) { return (w + 8 * q) % KS * 32 + 4 * (lx & 7); };
    auto load_m = [&](uint32_t rel) {
        const float* M = a.R + (int64_t)rel * a.rel_dim + D;
        Share s;
#pragma unroll
        for (int q = 0; q < BLOCKS; ++q) {
            const int e = me(q), d = md(q);
#pragma unroll
            for (int i = 0; i < 4; ++i) s.m[q][i] = ld4(M + (e + i < D && d < D ? (e + i) * D + d : 0));
        }
        return s;
    };
    // its parts to LDS; zeros outside the matrix
    auto store_parts = [&](const Share& s, auto large) {
#pragma unroll
        for (int q = 0; q < BLOCKS; ++q) {
            const int e = me(q), d = md(q);
            if (w + 8 * q >= KS * KS) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 x = e + i < D && d < D ? s.m[q][i] : f4(0.f);
                const Split2 lo = split2<large.value>(x.x, x.y), hi = split2<large.value>(x.z, x.w);
                uint16_t* to = Ms + unit_at(e + i, d);
#pragma unroll
                for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2*>(to + p * PART) = make_uint2(lo.p[p], hi.p[p]);
            }
        }
    };
    auto store_m = [&](const Share& s) {
        float m = 0.f;
#pragma unroll
        for (int q = 0; q < BLOCKS; ++q) {
#pragma unroll
            for (int i = 0; i < 4; ++i) m = fmaxf(m, magnitude(s.m[q][i]));
        }
        if (__any(is_large(m))) store_parts(s, std::true_type());
        else store_parts(s, std::false_type());
    };
    // right operands: K along the rows of M (N M^T) ...
    auto along_rows = [&](int ct, int ks) {
        const int l16 = lx & 15, quad = lx >> 4;
        const int swz = unit_at(l16, 0) & 127;  // the permutation of row l16 (and of every row 16 further on)
        const uint16_t* p = Ms + 128 * (16 * ct + l16) + ((32 * ks + 8 * quad) ^ swz);
        Split8 b;
#pragma unroll
        for (int q = 0; q < 3; ++q) b.p[q] = *reinterpret_cast<const bf16x8*>(p + q * PART);
        return b;
    };
    // ... and down its columns (V M): the transposing read gives a lane of sixteen four rows of its column; lane l16 names row l16 / 4
    // and columns 4 (l16 % 4) .. of them
    auto down_columns = [&](int ct, int ks) {
        const int l16 = lx & 15, quad = lx >> 4;
        const int tr0 = unit_at(8 * quad + (l16 >> 2), 0) & 127, tr1 = unit_at(8 * quad + 4 + (l16 >> 2), 0) & 127;
        typedef short shortx4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) shortx4* lds4;
        const int col = 16 * ct + 4 * (l16 & 3), row = 32 * ks + 8 * quad + (l16 >> 2);
        uint16_t* p0 = Ms + 128 * row + ((col & ~7) ^ tr0) + (col & 4);
        uint16_t* p1 = Ms + 128 * (row + 4) + ((col & ~7) ^ tr1) + (col & 4);
        Split8 b;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p0 + q * PART));
            const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p1 + q * PART));
            b.p[q] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
        return b;
    };

    // left M or left M^T, sixteen columns after sixteen, so that few accumulators are alive; a step's right operand is read while the
    // one before is multiplied
    auto product = [&](const Split8 (&left)[KS], auto right, auto out) {
        Split8 b = right(0, 0);
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            floatx4 big = {0.f, 0.f, 0.f, 0.f}, small = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const Split8 next = right(ks + 1 < KS ? ct : ct + 1 < NT ? ct + 1 : 0, ks + 1 < KS ? ks + 1 : 0);
                __builtin_amdgcn_sched_barrier(0);
                mfma_split(left[ks], b, big, small);
                b = next;
            }
            out(ct, big + small);
        }
    };

    floatx4 sum[NT];  // gradient rows of this wave's corrupting rows
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) sum[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
    float loss = 0.f;
    const int q4 = ((tid >> 2) & 1) + 2 * ((tid >> 3) & 1), x4 = tid & 3;  // what sum16x4 leaves this lane: row 4 quad + q4, positive x4
    const int jq = 16 * w + 4 * quad + q4;
    TransrBlock u = units[min(first, max(n_units - 1, 0))];
    Share share = load_m(u.rel);
    for (int e = first; e < end; ++e) {
        const TransrBlock next = units[min(e + 1, n_units - 1)];
        const int n = u.n;
        lds_barrier();  // the unit before is done with LDS
        again();
        store_m(share);
        for (int x = tid; x < n * (W / 4); x += UT) {  // o rows, zeros past column D
            const int m = x / (W / 4), d = 4 * (x % (W / 4));
            st4(Os + m * W + d, d < D ? ld4(a.O + (int64_t)(u.off + m) * D + d) : f4(0.f));
        }
        lds_barrier();
        // from here to the next barrier every wave goes its own way
        if (active) {
            floatx4 p[NT], vsum[NT];
            // (zeros past column D, also where a row with an infinity has met the zeros there)
            again();
            product(nf, along_rows, [&](int ct, floatx4 x) { p[ct] = 16 * ct + l16 < D ? x : floatx4{0.f, 0.f, 0.f, 0.f}; });
            float* W2 = Vs[w];  // [PB positives][16 rows]  2 W
            for (int m0 = 0; m0 < n; m0 += 4) {
                float r[4];
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    r[y] = 0.f;
                    if (m0 + y >= n) continue;
                    const float* po = Os + (m0 + y) * W + l16;
                    float ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ct = 0; ct < NT; ++ct) {
                        const float o = po[16 * ct];
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float d = o - p[ct][v];
                            ss[v] = fmaf(d, d, ss[v]);
                        }
                    }
                    r[y] = sum16x4(ss);
                }
                const float s = x4 == 0 ? r[0] : x4 == 1 ? r[1] : x4 == 2 ? r[2] : r[3];
                float w2 = 0.f;
                if (m0 + x4 < n && jq < rows) w2 = 2.f * w_and_loss<true>(a.gamma - s, a.wk, loss);
                W2[16 * (m0 + x4) + 4 * quad + q4] = w2;
            }
            wave_fence();
            // V and this wave's part of dL/do, four column tiles at a time, which leaves 64-bit sums the registers.  Of the sums over rows
            // every quarter of the wave gets those of one tile.
            static_assert(16 * PB <= 16 * UVP, "W where V is staged");
            auto v_and_go = [&](auto zero) {
                typedef decltype(zero) Sum;
                typedef Sum Sumx4 __attribute__((ext_vector_type(4)));
#pragma unroll
                for (int c0 = 0; c0 < NT; c0 += 4) {
                    Sumx4 acc[4] = {};
                    const int col = 16 * c0 + lane;
                    float* go = a.GOp + ((int64_t)(j0 / 16 + w) * a.b + u.off) * D + col;
#pragma unroll 1
                    for (int m = 0; m < n; ++m) {
                        const float4 ww = ld4(W2 + 16 * m + 4 * quad);
                        const Sum ws[4] = {ww.x, ww.y, ww.z, ww.w};
                        const float* po = Os + m * W + 16 * c0 + l16;
                        Sum g[4] = {};
#pragma unroll
                        for (int h = 0; h < 4; ++h) {
                            if (c0 + h >= NT) break;
                            const float o = po[16 * h];
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const Sum d = o - p[c0 + h][v];  // (a difference in 32 bits, exact where o is close to P)
                                acc[h][v] = __builtin_elementwise_fma(ws[v], d, (Sum)acc[h][v]);
                                g[h] = __builtin_elementwise_fma(-ws[v], d, g[h]);
                            }
                        }
                        const float x = (float)sum_quads(g);
                        if (col < D) go[(int64_t)m * D] = x;
                    }
#pragma unroll
                    for (int h = 0; h < 4; ++h)
                        if (c0 + h < NT) vsum[c0 + h] = __builtin_convertvector(acc[h], floatx4);
                }
            };
            // items of many positives: products and sums in 64 bits, as k_transr_dp has them (32 positives in 32 bits: 1.5 roundings in V, in
            // 64 bits 0.5; FB15k-sized 190 -> 194 us where that is done for every item)
            if (u.all > DP_FEW) v_and_go(0.);
            else v_and_go(0.f);
            wave_fence();
            float* V = a.V + ((int64_t)(c * a.g + e) * a.k + j0 + 16 * w + l16) * D + 8 * quad;
            const bool mine = 16 * w + l16 < rows;
            Split8 vf[KS];
#pragma unroll
            for (int k0 = 0; k0 < KS; k0 += 2) {  // two K steps at a time
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const int ct = 2 * k0 + h;
                    if (h >= 2 && k0 + 1 >= KS) break;
#pragma unroll
                    for (int v = 0; v < 4; ++v) Vs[w][(4 * quad + v) * UVP + 16 * h + l16] = ct < NT ? vsum[ct < NT ? ct : 0][v] : 0.f;
                }
                wave_fence();
#pragma unroll
                for (int ks = k0; ks < min(k0 + 2, KS); ++ks) {
                    const float* from = Vs[w] + l16 * UVP + 32 * (ks - k0) + 8 * quad;
                    const float4 lo = ld4(from), hi = ld4(from + 4);
                    if (mine && 32 * ks + 8 * quad < D) st4(V + 32 * ks, lo);
                    if (mine && 32 * ks + 8 * quad + 4 < D) st4(V + 32 * ks + 4, hi);
                    if (__any(is_large(fmaxf(magnitude(lo), magnitude(hi))))) vf[ks] = split_row<true>(lo, hi);
                    else vf[ks] = split_row<false>(lo, hi);
                }
                wave_fence();
            }
            again();
            product(vf, down_columns, [&](int ct, floatx4 x) { sum[ct] += x; });
            share = load_m(next.rel);  // (asked for before the product: D 128 221 -> 232 us, spills; D 100 the same)
        } else {
            share = load_m(next.rel);
        }
        u = next;
    }
    float* out = a.back_part + (((int64_t)seg * (a.b / a.g) + c) * a.k + j0 + 16 * w + 4 * quad) * D + l16;
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (16 * ct + l16 < D && 16 * w + 4 * quad + v < rows) out[(int64_t)v * D + 16 * ct] = sum[ct][v];
        }
    }
    loss = wave_sum(loss);
    if (lane == 0) part[w] = loss;
    __syncthreads();
    if (tid == 0) {
        float s = 0.f;
#pragma unroll
        for (int v = 0; v < 8; ++v) s += part[v];
        a.loss_part[blockIdx.x] = s * a.wk;
    }
}

}  // namespace
