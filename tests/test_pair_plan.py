"""How the backward launch of RotatE / TransE-L1 is cut (csrc/k_pair_plan.h), checked on the host over every row length
that kge_create accepts: each batch shape gets a cut, and the cut covers the chunk and stays inside the launch limits and
the buffers that kge_create sizes for it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_08532_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>

#include <initializer_list>

#include "k_pair_plan.h"

static int bad = 0;
#define CHECK(cond)                                                                                              \
    do {                                                                                                         \
        if (!(cond)) {                                                                                           \
            if (bad++ < 20) printf("cplx %d D %d b %d g %d k %d floats %lld: %s\n", cplx, D, b, g, k, (long long)floats, #cond); \
            return;                                                                                              \
        }                                                                                                        \
    } while (0)

static void check(bool cplx, int D, int b, int g, int k, int64_t floats) {
    const PairBwdPlan p = plan_pair_bwd(cplx, D, floats, b, k, g);
    const int NC = cplx ? D / 2 : D, chunks = b / g;
    CHECK(p.ti == 8 || p.ti == 16 || (p.ti == 32 && !cplx));
    CHECK(p.ng >= 1 && p.ng <= 64 && p.cpp >= 1 && p.ng * p.cpp <= 1024);
    CHECK((int64_t)p.n_col * p.cpp >= NC && (p.n_col - 1) * p.cpp < NC);
    CHECK(p.n_i == (g + p.ti - 1) / p.ti && p.i_parts >= 1 && p.i_parts <= p.n_i);
    CHECK(p.i_parts == p.n_i || p.ti == 16);                        // only tiles of 16 have the form that walks
    CHECK((int64_t)p.pj * p.tj >= k && (int64_t)(p.pj - 1) * p.tj < k && p.pj <= KGE_PAIR_MAX_PARTS);
    CHECK(p.i_parts == 1 || (int64_t)p.i_parts * chunks * k * D <= floats);
    CHECK((int64_t)p.i_parts * p.pj * chunks <= (int64_t)(b / 8 + chunks + 1) * KGE_PAIR_MAX_PARTS);  // loss sums
    const int block = pair_bwd_block(p.ti, p.ng, p.tj);
    CHECK(block >= p.ng && block % p.ng == 0);
    CHECK(pair_bwd_lds(cplx, p.ti, p.ng, p.cpp, block) <= 65536);
}

int main() {
    const int gs[] = {2, 3, 8, 17, 33, 100, 1000}, ks[] = {1, 2, 5, 64, 173, 1024}, chunks[] = {1, 3};
    for (int cplx = 0; cplx < 2; ++cplx)
        for (int D = cplx ? 8 : 4; D <= 1024; D += cplx ? 8 : 4)
            for (int g : gs)
                for (int k : ks)
                    for (int c : chunks)
                        for (int64_t floats : {(int64_t)1 << 40, (int64_t)3 * c * k * D, (int64_t)1})
                            check(cplx, D, c * g, g, k, floats);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_accepted_row_length_gets_a_cut(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout)
