// The work of one wave on row `row`: a positive (rows 0 .. b - 1) or a corrupting row (behind them).  In scope: MODEL, NV, the
// arguments `a`, row and lane.  Text that k_gather and gather_row include, not a function that both call: which product of a
// sum of products the compiler fuses depends on the function around it, that is the last bit of a positive's score, and the
// rank of a positive among candidates that tie with it hangs on that bit.  In this form k_gather rounds as it always has (as
// a function, 2 % of TransE-L2's and half of RESCAL's scores of positives came out one bit away).
    const int D = a.D;
    constexpr bool CPLX = (MODEL == KGE_COMPLEX || MODEL == KGE_ROTATE);
    const int nvec = CPLX ? D / 8 : D / 4;   // vectors (or re/im vector pairs) per row
    const int im_off = D / 2;                // float offset of the imaginary half

    if (row >= a.b + a.n_neg) return;
    const StepView sv = step_view(a.ids);

    if (row >= a.b) {  // ---- a corrupting row: copy it to staging
        const int j = row - a.b;
        const int64_t id = clamp_id(sv.neg[j], a.n_ent);
        const float* src = a.E + id * (int64_t)D;
        float* dst = a.Nst + (int64_t)j * D;
        float nn = 0.f;
        const int nv4 = D / 4;
        // every piece of the row is asked for before the first one is used (a load under a branch is waited for
        // where the branch ends: lanes past the row's end read its first piece instead)
        float4 xs[CPLX ? 2 * NV : NV];
#pragma unroll
        for (int it = 0; it < (CPLX ? 2 * NV : NV); ++it) xs[it] = ld4(src + 4 * (lane + it * 64 < nv4 ? lane + it * 64 : 0));
#pragma unroll
        for (int it = 0; it < (CPLX ? 2 * NV : NV); ++it) {
            const int v = lane + it * 64;
            if (v < nv4) {
                const float4 x = xs[it];
                float xv[4] = {x.x, x.y, x.z, x.w};
                if (a.bf16) {  // the product kernels round their operands to bf16: the norm is that of the rounded row
#pragma unroll
                    for (int e = 0; e < 4; ++e) xv[e] = round_bf16(xv[e]);
                }
                if (a.bf16) st4_bf16(a.Nbf + (int64_t)j * a.ld_bf + 4 * v, x.x, x.y, x.z, x.w);
                else st4(dst + 4 * v, x);
                nn += xv[0] * xv[0] + xv[1] * xv[1] + xv[2] * xv[2] + xv[3] * xv[3];
            }
        }
        if (MODEL == KGE_TRANSE_L2) {
            nn = wave_sum(nn);
            if (lane == 0) a.n_n2[j] = nn;
        }
        return;
    }

    // ---- a positive: rows a (kept entity), r, c (the entity that the negatives replace)
    if constexpr (MODEL == KGE_TRANSR) return;  // k_transr_phi does the positives (they need the matrix)
    const int i = row;
    const int64_t hid = clamp_id(sv.h[i], a.n_ent), tid = clamp_id(sv.t[i], a.n_ent);
    const int64_t rid = clamp_id(sv.r[i], a.n_rel);
    const bool head = sv.side == KGE_NEG_HEAD;
    const float* pa = a.E + (head ? tid : hid) * (int64_t)D;
    const float* pc = a.E + (head ? hid : tid) * (int64_t)D;
    const float* pr = a.R + rid * (int64_t)a.Dr;
    float* po = a.O + (int64_t)i * D;
    float acc = 0.f, on = 0.f;

    // all loads first, as for the corrupting rows.  L1 .. L6: the (up to six) 16-byte pieces that piece v of o needs
    float4 L1[NV], L2[NV], L3[NV], L4[NV], L5[NV], L6[NV];
#pragma unroll
    for (int it = 0; it < NV; ++it) {
        const int vs = lane + it * 64 < nvec ? lane + it * 64 : 0;
        if constexpr (MODEL == KGE_RESCAL) {
            L1[it] = ld4(po + 4 * vs); L2[it] = ld4(pc + 4 * vs);
        } else if constexpr (!CPLX) {
            L1[it] = ld4(pa + 4 * vs); L2[it] = ld4(pr + 4 * vs); L3[it] = ld4(pc + 4 * vs);
        } else {
            L1[it] = ld4(pa + 4 * vs); L2[it] = ld4(pa + im_off + 4 * vs);
            L3[it] = ld4(pc + 4 * vs); L4[it] = ld4(pc + im_off + 4 * vs);
            L5[it] = ld4(pr + 4 * vs);
            if (MODEL != KGE_ROTATE) L6[it] = ld4(pr + im_off + 4 * vs);
        }
    }
#pragma unroll
    for (int it = 0; it < NV; ++it) {
        const int v = lane + it * 64;
        if (v >= nvec) continue;
        if constexpr (MODEL == KGE_RESCAL) {
            // o_i = M_r^T h or M_r t is already in staging (k_rescal); the positive's score is o . c
            const float4 Oo = L1[it], Cc = L2[it];
            acc += Oo.x * Cc.x + Oo.y * Cc.y + Oo.z * Cc.z + Oo.w * Cc.w;
            if (a.bf16) {
                const float n0 = round_bf16(Oo.x), n1 = round_bf16(Oo.y), n2 = round_bf16(Oo.z), n3 = round_bf16(Oo.w);
                on += n0 * n0 + n1 * n1 + n2 * n2 + n3 * n3;
            }
        } else if constexpr (!CPLX) {
            const float4 A = L1[it], Rr = L2[it], Cc = L3[it];
            const float av[4] = {A.x, A.y, A.z, A.w}, rv[4] = {Rr.x, Rr.y, Rr.z, Rr.w}, cv[4] = {Cc.x, Cc.y, Cc.z, Cc.w};
            float ov[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (MODEL == KGE_DISTMULT) ov[e] = av[e] * rv[e];
                else ov[e] = head ? av[e] - rv[e] : av[e] + rv[e];
            }
            st4(po + 4 * v, make_float4(ov[0], ov[1], ov[2], ov[3]));
            if (a.bf16) st4_bf16(a.Obf + (int64_t)i * a.ld_bf + 4 * v, ov[0], ov[1], ov[2], ov[3]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (MODEL == KGE_DISTMULT) acc += ov[e] * cv[e];
                else if (MODEL == KGE_TRANSE_L1) acc += fabsf(ov[e] - cv[e]);
                else { const float u = ov[e] - cv[e]; acc += u * u; }
            }
            if (MODEL == KGE_TRANSE_L2 || a.bf16) {
                float nv[4] = {ov[0], ov[1], ov[2], ov[3]};
                if (a.bf16) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) nv[e] = round_bf16(nv[e]);
                }
                on += nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2] + nv[3] * nv[3];
            }
        } else {
            const float4 Are = L1[it], Aim = L2[it];
            const float4 Cre = L3[it], Cim = L4[it];
            const float are[4] = {Are.x, Are.y, Are.z, Are.w}, aim[4] = {Aim.x, Aim.y, Aim.z, Aim.w};
            const float cre[4] = {Cre.x, Cre.y, Cre.z, Cre.w}, cim[4] = {Cim.x, Cim.y, Cim.z, Cim.w};
            float rre[4], rim[4];
            if (MODEL == KGE_ROTATE) {
                const float4 Th = L5[it];
                const float th[4] = {Th.x, Th.y, Th.z, Th.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) sincosf(th[e], &rim[e], &rre[e]);
            } else {
                const float4 Rre = L5[it], Rim = L6[it];
                rre[0] = Rre.x; rre[1] = Rre.y; rre[2] = Rre.z; rre[3] = Rre.w;
                rim[0] = Rim.x; rim[1] = Rim.y; rim[2] = Rim.z; rim[3] = Rim.w;
            }
            float ore[4], oim[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float ri = head ? -rim[e] : rim[e];  // head corruption: o = t * conj(r)
                ore[e] = are[e] * rre[e] - aim[e] * ri;
                oim[e] = are[e] * ri + aim[e] * rre[e];
            }
            st4(po + 4 * v, make_float4(ore[0], ore[1], ore[2], ore[3]));
            st4(po + im_off + 4 * v, make_float4(oim[0], oim[1], oim[2], oim[3]));
            if (a.bf16) {
                st4_bf16(a.Obf + (int64_t)i * a.ld_bf + 4 * v, ore[0], ore[1], ore[2], ore[3]);
                st4_bf16(a.Obf + (int64_t)i * a.ld_bf + im_off + 4 * v, oim[0], oim[1], oim[2], oim[3]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (MODEL == KGE_COMPLEX) acc += ore[e] * cre[e] + oim[e] * cim[e];
                else {
                    const float qre = ore[e] - cre[e], qim = oim[e] - cim[e];
                    acc += sqrtf(qre * qre + qim * qim);
                }
            }
        }
    }
    acc = wave_sum(acc);
    if (MODEL == KGE_TRANSE_L2) on = wave_sum(on);
    if (lane == 0) {
        float f;
        if (MODEL == KGE_TRANSE_L2) f = a.gamma - sqrtf(acc);
        else if (MODEL == KGE_TRANSE_L1 || MODEL == KGE_ROTATE) f = a.gamma - acc;
        else f = acc;
        a.fpos[i] = f;
        if (a.pos_out) a.pos_out[i] = f;
        if (a.rank_out) a.rank_out[i] = 1;
        if (MODEL == KGE_TRANSE_L2) {
            a.o_n2[i] = on;
            a.inv_dpos[i] = acc > 0.f ? 1.f / sqrtf(acc) : 0.f;
        }
        // positive part of the logistic loss (Sec. 2, y = +1) and its derivative
        const float invb = 1.f / (float)a.b;
        const float e = expf(-fabsf(f));
        a.row_loss[i] = (fmaxf(-f, 0.f) + log1pf(e)) * invb;
        a.cpos[i] = -((f >= 0.f ? e : 1.f) / (1.f + e)) * invb;
    }
