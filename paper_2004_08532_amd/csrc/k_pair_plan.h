// How the backward launch of RotatE / TransE-L1 (k_pair.hip) is cut for batches of one shape.  Host code only.
#pragma once
#include <stdint.h>

constexpr int KGE_PAIR_MAX_PARTS = 16;  // most partial rows of dL/do in the backward of RotatE / TransE-L1

struct PairBwdPlan { int b, k, g, ti, n_i, i_parts, pj, tj, n_col, cpp, ng; };

// Negatives per staged block of W: 48 KB of them, which is nearly always the whole range (one wait for the scores); bytes of
// LDS: W, later the sums of half of the thread groups.
inline int pair_bwd_block(int ti, int ng, int tj) {
    const int fit = 12288 / (ti + 4) / ng, need = (tj + ng - 1) / ng;
    return (need < fit ? need : fit) * ng;
}
inline int pair_bwd_lds(bool cplx, int ti, int ng, int cpp, int block) {
    const int w_floats = block * (ti + 4), sum_floats = ng / 2 * cpp * ti * (cplx ? 2 : 1);
    return 4 * (w_floats > sum_floats ? w_floats : sum_floats);
}

// How a backward launch is cut: the tile of positives, the ranges of coordinates and of negatives, and the size of a workgroup
// that an estimate of the running time likes best.  The estimate: rounds of workgroups (as many share a CU as registers
// and LDS let in) times the work of one (rounds of its thread groups over the negatives, staging of W, meeting of the
// groups' sums, a constant), plus the partial rows that are written here and added up by the chain launch.  Its constants
// were fitted to 11,000 measured launches of this kernel and the chain launch: 96 batch shapes (16 <= g <= 1000,
// 16 <= k <= 1024, 32 <= D <= 800), every cut that is tried here.  The cut it chooses takes 2.5 % longer than the best
// measured one on average, 16 % at most.
// At least one cut is always tried: tiles of 16 positives, whole rows (at most 1024 coordinates, so that one thread group
// of 1024 threads holds them).
inline PairBwdPlan plan_pair_bwd(bool cplx, int D, int64_t part_floats, int b, int k, int g) {
    const int NC = cplx ? D / 2 : D, chunks = b / g;
    const double term = cplx ? 13 : 6.6;  // issue slots per pair and coordinate
    PairBwdPlan best = {};
    double best_cost = 1e300;
    for (int ti = 8; ti <= (cplx ? 16 : 32); ti *= 2) {
        const int n_i = (g + ti - 1) / ti;
        const int64_t cap = part_floats / ((int64_t)chunks * k * D);
        const int i_parts = n_i <= cap ? n_i : (int)(cap > 1 ? cap : 1);
        if (i_parts < n_i && ti != 16) continue;
        const int walks = (n_i + i_parts - 1) / i_parts;
        const int cu_waves = cplx ? (ti == 8 ? 24 : 16) : (ti == 8 ? 28 : ti == 16 ? 24 : 16);  // what the registers let in
        for (int n_col = 1; n_col == 1 || (n_col <= 4 && NC >= 8 * n_col); ++n_col) {
            const int cpp = (NC + n_col - 1) / n_col;
            for (int threads = 512; threads <= 1024; threads *= 2) {
                int ng = threads / cpp;
                ng = ng > 64 ? 64 : ng;
                ng = ng > k ? k : ng;
                if (ng == 0) continue;
                const int waves = (ng * cpp + 63) / 64;
                for (int parts = 1; parts <= KGE_PAIR_MAX_PARTS; ++parts) {
                    if (parts > 1 && k < parts * ng) break;
                    const int tj = (k + parts - 1) / parts, pj = (k + tj - 1) / tj, iters = (tj + ng - 1) / ng;
                    const int lds = pair_bwd_lds(cplx, ti, ng, cpp, pair_bwd_block(ti, ng, tj)) + 2048;
                    const double wgs = (double)chunks * i_parts * n_col * pj;
                    int per_cu = cu_waves / waves;
                    if (per_cu > 163840 / lds) per_cu = 163840 / lds;
                    if (per_cu > (wgs + 255) / 256) per_cu = (int)((wgs + 255) / 256);
                    if (per_cu < 1) per_cu = 1;
                    const int rounds = (int)((wgs + 256 * per_cu - 1) / (256 * per_cu));
                    const int simd_waves = waves * per_cu > 4 ? waves * per_cu : 4;
                    double iter = (ti * term + 21) * simd_waves;
                    if (iter < 680) iter = 680;
                    int halvings = 0;
                    while (ng > 1 << halvings) ++halvings;
                    const double wg = walks * (iters * iter + 27000.0 * ((tj + 255) / 256) * ((ti + waves - 1) / waves) + 1060.0 * ti * halvings) + 34000;
                    const double bytes = ((i_parts > 1 ? 2.0 * i_parts * chunks * k : 0) + (pj > 1 ? 2.0 * pj * b : 0)) * D * 4;
                    const double cost = rounds * wg + bytes / 440;
                    if (cost < best_cost) {
                        best_cost = cost;
                        best = {b, k, g, ti, n_i, i_parts, pj, tj, n_col, cpp, ng};
                    }
                }
            }
        }
    }
    return best;
}
