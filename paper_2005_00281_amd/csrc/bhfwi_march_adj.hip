// bhfwi_march_adj.hip -- time-skewed adjoint march: T reverse steps of Eq. 6 (the
// exact transpose of the discrete forward) fused with the correlation of
// Eq. 7-8 and the illumination, one wave64 per tile and no barrier, on tiles
// clear of every PML layer.
//
// The march is that of the forward (bhfwi_march_fwd.hip): level t runs one row
// behind level t - 1; at march step s it takes row r = s - t of the adjoint
// state before its reverse step and finishes row q = r - 1.  The transposed
// step has the same reach: the adjoint velocities of row r (v_r) and row q
// (v_z) need the drivers (the transposed stress update of the adjoint stresses)
// of rows q and r, and the stresses of row q gather the products of rows q - 1,
// q and r.  Each level keeps 7 values of row q (old stresses and velocities, one
// product) and the stored velocities v^{n+1/2} its correlation still needs, and
// forms the drivers of row q again; the correlation sums of a row travel with it
// from level to level and are added to the accumulators once, when the row
// leaves the last level.  The stored velocities of the next march step are
// fetched one step ahead.
//
// What bounds it: memory.  64 shots of 276 x 4136 cells, six steps, beside the PML
// tiles: 10.3 GB in 1887 us (5.5 TB/s, three quarters of it reads; a copy moves
// 5.0) and 693e6 wave instructions (0.60 of one per compute unit and clock); 8 of
// the 92 B per cell-step are the stored velocities, which no blocking saves.  The
// PML tiles beside it end some 780 us later and bound the block.  12 of those
// shots, 1250 steps: gradient 265.1 ms, 315.7 with all tiles in LDS.  Over 39
// surveys the adjoint was 1.05 times as fast as on LDS tiles of six steps, from
// 0.93 (19 shots of 211 x 2417 cells) to 1.17.  T = 8 spills and is not built: an
// adjoint of eight steps per launch keeps its LDS tiles.
//
// X selects the optional outputs of bhfwi_tb_adj.hip: bit 0 the density
// correlation, bit 1 the pseudo-Hessian diagonal, bit 2 the wavelet record.
#pragma once
#include "bhfwi_internal.h"
#include "bhfwi_march_fwd.hip"

namespace bhfwi {
namespace march {

template <int T, int X>
__global__ void __launch_bounds__(64, 2)
k_adj_march(const ShotDev* __restrict__ shots, const int4* __restrict__ work, int nwork, int map,
            int tz, int n_hi, const float* __restrict__ lam, const float* __restrict__ mu,
            const float* __restrict__ rho, const int* __restrict__ rec_k,
            const float* __restrict__ resid, const float* __restrict__ pml_r,
            const float* __restrict__ ain, float* __restrict__ aout,
            const float* __restrict__ hist_hi, long long hist_stride, float* __restrict__ acc,
            float* __restrict__ acc_rho, float* __restrict__ acc_h, float* __restrict__ wgrad,
            long long cells_total)
{
#pragma clang fp contract(off)
    static_assert(T >= 1 && T <= kRing, "ring too small");
    constexpr bool RHO = (X & 1) != 0, HES = (X & 2) != 0, WAV = (X & 4) != 0;
    __shared__ float L[kRing][kCoef][64];
    __shared__ float Lres[T][64];  // residual/3 of this lane's receiver, per step

    const int wg = xcd_chunk(blockIdx.x, nwork, map);
    if (wg >= nwork) return;
    const int4 wk = work[wg];  // shot, first owned axial row, radial rows [z, w)
    const ShotDev& S = shots[wk.x];
    // levels t < t0 lie past the end of this shot's record: its state is zero
    // there and nothing is correlated
    const int t0 = max(0, n_hi - (S.nt - 1));
    if (t0 >= T) return;

    const int lane = threadIdx.x;
    const int NR = S.NR, NZ = S.NZ;
    const long long cells = (long long)NR * NZ;
    const int i0 = wk.z, i1 = wk.w;
    const int k = wk.y - T + lane;  // interior tiles: the owned lanes and their halo lie in the grid
    const bool own = lane >= T && lane < T + tz;
    const unsigned kb = 4u * (unsigned)min(k, NZ - 1);
    const unsigned kmb = 4u * (unsigned)min(k + (lane == 63), NZ - 1);
    // the correlation of the owned cells reads one column around them only
    const unsigned khb = 4u * (unsigned)min(max(k, wk.y - 1), wk.y + tz);
    const float dt = S.dt, idr = S.inv_dr, idz = S.inv_dz;

    const float* __restrict__ Ai = ain + S.ast_off;
    float* __restrict__ Ao = aout + S.ast_off;
    const float* __restrict__ rRt = pml_r + S.pml_r_off + 4 * NR;  // 1/(2 r) at R nodes
    const float* __restrict__ rZt = rRt + NR;                      // and at C and Z nodes
    const float* __restrict__ lam_m = lam + S.model_off;
    const float* __restrict__ mu_m = mu + S.model_off;
    const float* __restrict__ rho_m = rho + S.model_off;
    const float* __restrict__ h_s = hist_hi + S.cell_off;
    float* __restrict__ g_s = acc + S.cell_off;
    const int rowB = 4 * NZ, rowM = 4 * (int)S.model_ld;

#pragma unroll
    for (int q = 0; q < kRing * kCoef; ++q) (&L[0][0][0])[q * 64 + lane] = 0.f;
    {
        float rsum[T];
#pragma unroll
        for (int t = 0; t < T; ++t) rsum[t] = 0.f;
        if (i0 == 0)
            for (int r = 0; r < S.nrec; ++r)
                if (rec_k[S.rec_off + r] == k) {
#pragma unroll
                    for (int t = 0; t < T; ++t)
                        if (t >= t0)
                            rsum[t] += resid[S.trace_off + (long long)r * S.nt + (n_hi - t)];
                }
#pragma unroll
        for (int t = 0; t < T; ++t) Lres[t][lane] = rsum[t] * (1.0f / 3.0f);
    }

    struct Row {
        float vr, vz, trr, ttt, tzz, trz, gR;
    };
    float o_trr[T], o_ttt[T], o_tzz[T], o_trz[T], o_vz[T], o_avr[T];
    float oZR[T];                    // product of row q - 1 that row q gathers
    float hvr[T], hvz[T];            // stored v_r of row q, v_z of row q - 1
    float pvr[T], pvz[T];            // fetched: v_r of row r, v_z of row q of the next step
    float gl[T], gm[T], gs[T], ge[T];  // sums of the row the level takes next
    float oR[T], gZ[T], hL[T], hM[T], wsa[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        o_trr[t] = o_ttt[t] = o_tzz[t] = o_trz[t] = o_vz[t] = o_avr[t] = 0.f;
        oZR[t] = 0.f;
        hvr[t] = hvz[t] = pvr[t] = pvz[t] = 0.f;
        gl[t] = gm[t] = gs[t] = ge[t] = 0.f;
        oR[t] = gZ[t] = hL[t] = hM[t] = wsa[t] = 0.f;
    }
    float rRs[T + 1], rZs[T + 1], p_rR = 0.f, p_rZ = 0.f;
#pragma unroll
    for (int t = 0; t <= T; ++t) rRs[t] = rZs[t] = 0.f;
    const int sbeg = max(0, i0 - T), send = i1 - 1 + T;
    long long hstr = hist_stride;
    Row P{};
    float p_lam, p_mu, p_muk, p_rho, mu_prev = 0.f, muk_prev = 0.f, rho_prev = 1.f, bZ_prev = 0.f;
    auto fetch = [&](int i) {  // adjoint state and model of row i (inside the grid: i <= send + 1)
        const unsigned c = kb + (unsigned)(i * rowB), m = kb + (unsigned)(i * rowM);
        p_rR = rRt[i];
        p_rZ = rZt[i];
        P.vr = ldrow(Ai, c);
        P.vz = ldrow(Ai + cells, c);
        P.trr = ldrow(Ai + 2 * cells, c);
        P.ttt = ldrow(Ai + 3 * cells, c);
        P.tzz = ldrow(Ai + 4 * cells, c);
        P.trz = ldrow(Ai + 5 * cells, c);
        p_lam = ldrow(lam_m, m);
        p_mu = ldrow(mu_m, m);
        p_muk = ldrow(mu_m, kmb + (unsigned)(i * rowM));
        p_rho = ldrow(rho_m, m);
    };
    // stored velocities that level t takes in march step s: v_r of row s - t and
    // v_z of row s - t - 1 at step n_hi - t.  GEN: rows below the axis read row 0
    // instead (their sums are never written); levels past the record take zeros.
    auto fetch_hist = [&](int s, int t, auto GENC) {
        constexpr bool GEN = decltype(GENC)::value != 0;
        const int r = GEN ? max(s - t, 0) : s - t, q = GEN ? max(s - t - 1, 0) : s - t - 1;
        const float* hv = h_s - (long long)t * hstr;
        const float a = ldrow(scalar_row(hv + (long long)r * NZ), khb);
        const float b = ldrow(scalar_row(hv + cells_total + (long long)q * NZ), khb);
        pvr[t] = GEN && t < t0 ? 0.f : a;
        pvz[t] = GEN && t < t0 ? 0.f : b;
    };
    if (sbeg >= 1) {
        mu_prev = ldrow(mu_m, kb + (unsigned)((sbeg - 1) * rowM));
        muk_prev = ldrow(mu_m, kmb + (unsigned)((sbeg - 1) * rowM));
        rho_prev = ldrow(rho_m, kb + (unsigned)((sbeg - 1) * rowM));
    }
    fetch(sbeg);
#pragma unroll
    for (int t = 0; t < T; ++t) fetch_hist(sbeg, t, IntC<1>{});

    auto step = [&](int s, auto GENC) {
        constexpr bool GEN = decltype(GENC)::value != 0;
        Row in = P;
        in.gR = 0.f;
        if constexpr (GEN) {
            if (s == 0) in.vr = in.trz = 0.f;  // nodes on the axis
        }
        // the last lane's driver reaches the lane below it in the same step: it takes
        // the column above it from memory (after the exchange: all lanes take part)
        float mu_kp = from_lane_above(p_mu), mu_mkp = from_lane_above(mu_prev);
        mu_kp = lane == 63 ? p_muk : mu_kp;
        mu_mkp = lane == 63 ? muk_prev : mu_mkp;
        const Coef cf = coefs(dt, p_lam, p_mu, p_rho, mu_prev, rho_prev, mu_kp, mu_mkp,
                              !GEN || s >= 1);
        muk_prev = p_muk;
        mu_prev = p_mu;
        rho_prev = p_rho;
#pragma unroll
        for (int t = T; t > 0; --t) {
            rRs[t] = rRs[t - 1];
            rZs[t] = rZs[t - 1];
        }
        rRs[0] = p_rR;
        rZs[0] = p_rZ;
        if (s < send) fetch(s + 1);  // uniform
        // the accumulators of the row that leaves the last level in this step
        const int qo = s - T;
        const unsigned co = kb + (unsigned)(qo * rowB);
        const bool out = !GEN || (qo >= i0 && qo < i1);
        float a_l = 0.f, a_m = 0.f, a_s = 0.f, a_e = 0.f, a_R = 0.f, a_Z = 0.f, a_hl = 0.f,
              a_hm = 0.f;
        if (out) {
            a_l = ldrow(g_s, co);
            a_m = ldrow(g_s + cells_total, co);
            a_s = ldrow(g_s + 2 * cells_total, co);
            a_e = ldrow(g_s + 3 * cells_total, co);
            if constexpr (RHO) {
                a_R = ldrow(acc_rho + S.cell_off, co);
                a_Z = ldrow(acc_rho + S.cell_off + cells_total, co);
            }
            if constexpr (HES) {
                a_hl = ldrow(acc_h + S.cell_off, co);
                a_hm = ldrow(acc_h + S.cell_off + cells_total, co);
            }
        }
        const int sn = min(s + 1, send);  // the last step fetches its own rows again
        asm volatile("" : "+s"(hstr));  // history rows are addressed as they come
        __builtin_amdgcn_sched_barrier(0);
        auto ring = [&](int r) {
            const float(*Lq)[64] = L[r & (kRing - 1)];
            return Coef{Lq[0][lane], Lq[1][lane], Lq[2][lane], Lq[4][lane], Lq[3][lane]};
        };
        Coef nx = Coef{cf.cl, cf.c2m, cf.bR, 0.f, cf.mS};
        nx.bZ = bZ_prev;  // of row s - 1
        // sums handed to the next level (zero for a row that enters)
        float cgl = 0.f, cgm = 0.f, cgs = 0.f, cge = 0.f, cgZ = 0.f, chL = 0.f, chM = 0.f;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int r = s - t, q = r - 1;
            const Coef c = nx;
            nx = ring(q);  // row q: this level's old row, the next level's new one
            const float vr1 = pvr[t], vz0 = pvz[t];
            fetch_hist(sn, t, GENC);
            __builtin_amdgcn_sched_barrier(0);
            const float rR = rRs[t], rRq = rRs[t + 1], rZr = rZs[t], rZ = rZs[t + 1];
            // A: residual, drivers of the transposed stress update at row r
            if constexpr (GEN) {
                const float v = r == 0 ? Lres[t][lane] : 0.f;
                in.trr += v;
                in.ttt += v;
                in.tzz += v;
            }
            const float sa = in.trr + in.ttt + in.tzz;
            if constexpr (WAV && GEN) wsa[t] = r == 0 ? sa : wsa[t];
            const float e0 = c.cl * sa;
            const float Err = fmaf(in.trr, c.c2m, e0), Ett = fmaf(in.ttt, c.c2m, e0);
            const float Ez = c.mS * in.trz;
            // the drivers of row q, formed again rather than kept
            const float saq = o_trr[t] + o_ttt[t] + o_tzz[t], e0q = nx.cl * saq;
            const float Errq = fmaf(o_trr[t], nx.c2m, e0q), Ettq = fmaf(o_ttt[t], nx.c2m, e0q);
            const float Ezzq = fmaf(o_tzz[t], nx.c2m, e0q);
            const float Ezq = nx.mS * o_trz[t];
            // B: Eq. 7-8 at row q with the strain rates of v^{n+1/2} and dJ/dtau^{n+1}
            const float vz_km = from_lane_below(vz0), vr_kp = from_lane_above(hvr[t]);
            const float dvr = vr1 - hvr[t], dvz = vz0 - vz_km;
            const float ur = hvr[t] + vr1, uz = vz_km + vz0;  // twice the C-node means
            const float err = idr * dvr, ett = ur * rZ, ezz = idz * dvz;
            const float dv = fmaf(idz, dvz, fmaf(idr, dvr, ett));
            const float es = fmaf(idr, vz0 - hvz[t], (vr_kp - hvr[t]) * idz);
            {
                const float n_l = fmaf(dv, saq, gl[t]);
                const float n_m =
                    fmaf(err, o_trr[t], fmaf(ett, o_ttt[t], fmaf(ezz, o_tzz[t], gm[t])));
                const float n_s = fmaf(es, o_trz[t], gs[t]);
                const float n_e = fmaf(ur, ur, fmaf(uz, uz, ge[t]));
                gl[t] = cgl;
                gm[t] = cgm;
                gs[t] = cgs;
                ge[t] = cge;
                cgl = n_l;
                cgm = n_m;
                cgs = n_s;
                cge = n_e;
            }
            // formed here, not when the row leaves: what they are formed from goes
            asm volatile("" : "+v"(cgl), "+v"(cgm), "+v"(cgs), "+v"(cge));
            if constexpr (HES) {
                const float e2 = GEN && q < 1 ? 0.f : es;
                const float n_l = fmaf(3.0f * dv, dv, hL[t]);
                const float n_m = hM[t] + fmaf(4.0f, fmaf(ezz, ezz, fmaf(err, err, ett * ett)),
                                               e2 * e2);
                hL[t] = chL;
                hM[t] = chM;
                chL = n_l;
                chM = n_m;
                asm volatile("" : "+v"(chL), "+v"(chM));
            }
            // transposed stress update into a_v, then the transposed velocity update
            float dar = fmaf(idr, Errq - Err, Ettq * rZ);
            dar = fmaf(rZr, Ett, dar);
            dar = fmaf(idz, from_lane_below(Ez) - Ez, dar);
            const float daz = fmaf(idz, Ezzq - from_lane_above(Ezzq), (Ezq - Ez) * idr);
            const float avr = in.vr + dar, avz = o_vz[t] + daz;
            if constexpr (RHO) {
                in.gR = fmaf(dar, vr1, in.gR);
                const float n_z = fmaf(daz, vz0, gZ[t]);
                gZ[t] = cgZ;
                cgZ = n_z;
                asm volatile("" : "+v"(in.gR), "+v"(cgZ));
            }
            const float W1 = c.bR * avr, W2 = c.bZ * avz, W1q = nx.bR * o_avr[t];
            const float U0 = W1q * idr, U1 = W1 * idr, H0 = W1q * rRq, H1 = W1 * rR;
            const float ZH = W2 * rZ;
            // C: gathered into a_tau of row q
            Row o;
            o.trr = o_trr[t] + (((H0 + U0) - U1) + H1);
            o.ttt = o_ttt[t] - (H0 + H1);
            o.tzz = fmaf(idz, fmaf(-avz, c.bZ, from_lane_below(W2)), o_tzz[t]);
            o.trz = o_trz[t] + fmaf(idz, fmaf(o_avr[t], nx.bR, -from_lane_above(W1q)),
                                    fmaf(-idr, W2, ZH));
            o.trz += oZR[t];
            if constexpr (GEN) o.trz = q < 1 ? 0.f : o.trz;
            o.vr = o_avr[t];
            o.vz = avz;
            o.gR = oR[t];
            o_trr[t] = in.trr;
            o_ttt[t] = in.ttt;
            o_tzz[t] = in.tzz;
            o_trz[t] = in.trz;
            o_vz[t] = in.vz;
            o_avr[t] = avr;
            oZR[t] = fmaf(idr, W2, ZH);
            hvr[t] = vr1;
            hvz[t] = vz0;
            oR[t] = in.gR;
            in = o;
        }
        // row s enters the ring once its slot's last reader (row s - T) is done
        float(*Ls)[64] = L[s & (kRing - 1)];
        Ls[0][lane] = cf.cl;
        Ls[1][lane] = cf.c2m;
        Ls[2][lane] = cf.bR;
        Ls[3][lane] = cf.mS;
        Ls[4][lane] = bZ_prev;
        bZ_prev = cf.bZ;
        if (out && own) {
            if (!GEN || qo >= 1) {
                strow(Ao, co, in.vr);
                strow(Ao + 5 * cells, co, in.trz);
                strow(g_s + 2 * cells_total, co, fmaf(dt, cgs, a_s));
                if constexpr (RHO) strow(acc_rho + S.cell_off, co, a_R + in.gR);
            }
            strow(Ao + cells, co, in.vz);
            strow(Ao + 2 * cells, co, in.trr);
            strow(Ao + 3 * cells, co, in.ttt);
            strow(Ao + 4 * cells, co, in.tzz);
            strow(g_s, co, fmaf(dt, cgl, a_l));
            strow(g_s + cells_total, co, fmaf(2.0f * dt, cgm, a_m));
            strow(g_s + 3 * cells_total, co, fmaf(0.25f * dt, cge, a_e));
            if constexpr (RHO) strow(acc_rho + S.cell_off + cells_total, co, a_Z + cgZ);
            if constexpr (HES) {
                strow(acc_h + S.cell_off, co, fmaf(dt * dt, chL, a_hl));
                strow(acc_h + S.cell_off + cells_total, co, fmaf(dt * dt, chM, a_hm));
            }
        }
    };
    // steady steps: past the axis row at every level, and the row that leaves is owned
    const int fast0 = t0 > 0 ? send + 1 : max(i0 + T, T + 1);
    int s = sbeg;
    while (s <= send) {
        while (s >= fast0 && s + 1 <= send) {  // two steps: registers swap roles
            step(s, IntC<0>{});
            step(s + 1, IntC<0>{});
            s += 2;
        }
        if (s > send) break;
        step(s, IntC<1>{});
        ++s;
    }
    if constexpr (WAV) {
        // the tile that owns row 0 and the source cell's lane
        if (i0 == 0 && own && k == S.src_k)
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (t >= t0) wgrad[S.wave_off + (n_hi - t)] = S.src_scale * wsa[t];
    }
}

}  // namespace march
}  // namespace bhfwi
