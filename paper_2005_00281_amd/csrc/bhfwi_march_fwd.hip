// bhfwi_march_fwd.hip -- time-skewed forward march (Method section, Eq. 2): T
// time steps per launch with one wave64 per tile and no barrier, on tiles clear
// of every PML layer.
//
// A wave owns a strip of axial columns (lane = axial row of the grid, T halo
// lanes on each side) and the radial rows [i0, i1) of them.  It marches outwards
// in radius; level t of the block (0 .. T-1) runs one row behind level t - 1:
// at march step s level t takes row r = s - t of the state before its time step
// and finishes row q = r - 1, which is at once the row that level t + 1 takes.
// A staggered step reads one row on either side, so everything a level has to
// remember between two march steps is seven values per lane (the old stresses
// and v_z of row q, the new v_r of row q and the new v_z of row q - 1): the
// whole block lives in registers, radial neighbours are the wave's own
// registers and axial neighbours its lanes (DPP wavefront shifts).  The medium
// coefficients of a row are set up once, when the row enters, and wait in a
// ring of 8 rows in LDS for the levels that follow (private to the wave: no
// barrier).  The next row is loaded while the current one is worked on.
//
// Against the LDS tiles of bhfwi_tb_fwd.hip, which hold a whole tile and
// recompute a halo of T rows above and below it, the march recomputes halo
// columns only (and T rows below a tile that does not start at the axis), has
// no barrier to wait at and exchanges nothing between waves.  Tiles that reach a
// PML layer stay with the LDS tiles: the memories would double the registers a
// level keeps.
//
// What bounds it: vector issue and memory together.  64 shots of 276 x 4136
// cells, eight steps, beside the PML tiles: 4.73 GB in 1042 us (4.5 TB/s where a
// copy moves 5.0) and 485e6 wave instructions (0.76 of one per compute unit and
// clock); with the stored velocities 8.94 GB in 2065 us (4.3 TB/s).  12 of those
// shots, 1250 steps: 52.0 ms, 72.9 in LDS tiles.
//
// The product-sums are explicit (contraction off), fused as the compiler fuses
// them in the LDS tiles clear of the layers; the PML form adds its memories
// between them and rounds on its own.  So which form computed a cell shows in its
// value at FP32 rounding: moving rows between them moved modelled traces by 1.6e-6
// (relative L2).
#pragma once
#include "bhfwi_internal.h"
#include "bhfwi_kernels.hip"

namespace bhfwi {
namespace march {

constexpr int kRing = 8;   // rows of coefficients kept in LDS
constexpr int kCoef = 5;   // coefficients per cell

__device__ inline float ldrow(const float* __restrict__ row, unsigned byte_off)
{
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + byte_off);
}
__device__ inline void strow(float* __restrict__ row, unsigned byte_off, float v)
{
    *reinterpret_cast<float*>(reinterpret_cast<char*>(row) + byte_off) = v;
}

// A row address that is the same in every lane, kept in scalar registers where
// it is used (not folded with the lane's offset into a vector address).
__device__ inline unsigned long long scalar_addr(unsigned long long v)
{
    int lo = __builtin_amdgcn_readfirstlane((int)v);
    int hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
    asm volatile("" : "+s"(lo), "+s"(hi));
    return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}
__device__ inline const float* scalar_row(const float* p)
{
    return reinterpret_cast<const float*>(scalar_addr(reinterpret_cast<unsigned long long>(p)));
}
__device__ inline float* scalar_row(float* p)
{
    return reinterpret_cast<float*>(scalar_addr(reinterpret_cast<unsigned long long>(p)));
}

// Medium coefficients of one row, from the model values of the row and the
// row below it; up: the row has one below it (v_r and tau_rz vanish on the
// axis).  mu_kp and mu_mkp: the rigidities of the column above.  The last
// lane's bZ lacks its neighbour: only its own v_z takes it, which is halo.
struct Coef {
    float cl, c2m, bR, bZ, mS;
};
__device__ inline Coef coefs(float dt, float lam, float mu, float rho, float mu_m, float rho_m,
                             float mu_kp, float mu_mkp, bool up)
{
    Coef c;
    c.cl = dt * lam;
    c.c2m = dt * 2.0f * mu;
    c.bR = up ? dt * 2.0f * rcp(rho_m + rho) : 0.f;
    c.bZ = dt * 2.0f * rcp(rho + from_lane_above(rho));
    c.mS = up ? dt * mu_harm(mu_m, mu, mu_mkp, mu_kp) : 0.f;
    return c;
}

// 1/(2 r) of every radial row, behind the shot's radial PML table: at the R
// nodes (0 on the axis), then at the C and Z nodes; the values the LDS tiles
// form for themselves.  One workgroup per shot.
__global__ void k_radii(const ShotDev* __restrict__ shots, float* __restrict__ pml_r)
{
    const ShotDev& S = shots[blockIdx.x];
    float* __restrict__ t = pml_r + S.pml_r_off + 4 * S.NR;
    for (int i = threadIdx.x; i < S.NR; i += blockDim.x) {
        t[i] = i >= 1 ? 0.5f * rcp(i * S.dr) : 0.f;
        t[S.NR + i] = 0.5f * rcp((i + 0.5f) * S.dr);
    }
}

template <int T, int HIST>
__global__ void __launch_bounds__(64, 3)
k_fwd_march(const ShotDev* __restrict__ shots, const int4* __restrict__ work, int nwork, int map,
            int tz, int n0, const float* __restrict__ lam, const float* __restrict__ mu,
            const float* __restrict__ rho, const float* __restrict__ wavelet,
            const int* __restrict__ rec_k, const float* __restrict__ pml_r,
            const float* __restrict__ sin, float* __restrict__ sout, float* __restrict__ traces,
            float* __restrict__ hist, long long hist_stride, long long cells_total)
{
#pragma clang fp contract(off)
    static_assert(T >= 1 && T <= kRing, "ring too small");
    __shared__ float L[kRing][kCoef][64];

    const int wg = xcd_chunk(blockIdx.x, nwork, map);
    if (wg >= nwork) return;
    const int4 wk = work[wg];  // shot, first owned axial row, radial rows [z, w)
    const ShotDev& S = shots[wk.x];
    if (n0 >= S.nt) return;

    const int lane = threadIdx.x;
    const int NR = S.NR, NZ = S.NZ;
    const long long cells = (long long)NR * NZ;
    const int i0 = wk.z, i1 = wk.w;
    const int k = wk.y - T + lane;  // interior tiles: the owned lanes and their halo lie in the grid
    const bool own = lane >= T && lane < T + tz;
    const unsigned kb = 4u * (unsigned)min(k, NZ - 1);  // byte offset of the lane in a row
    const float dt = S.dt, idr = S.inv_dr, idz = S.inv_dz;

    // plane bases; a row is addressed by a 32-bit byte offset per lane (the host
    // keeps planes and model windows of 2^31 bytes or more off the march)
    const float* __restrict__ Fi = sin + S.fst_off;
    float* __restrict__ Fo = sout + S.fst_off;
    const float* __restrict__ rRt = pml_r + S.pml_r_off + 4 * NR;  // 1/(2 r) at R nodes
    const float* __restrict__ rZt = rRt + NR;                      // and at C and Z nodes
    const float* __restrict__ lam_m = lam + S.model_off;
    const float* __restrict__ mu_m = mu + S.model_off;
    const float* __restrict__ rho_m = rho + S.model_off;
    const int rowB = 4 * NZ, rowM = 4 * (int)S.model_ld;
    float* const tr_s = traces ? traces + S.trace_off : nullptr;
    float* const h_s = HIST ? hist + S.cell_off : nullptr;
    float wv[T];  // source samples of the block's steps
#pragma unroll
    for (int t = 0; t < T; ++t)
        wv[t] = (i0 == 0 && n0 + t < S.nt) ? wavelet[S.wave_off + n0 + t] : 0.f;

#pragma unroll
    for (int q = 0; q < kRing * kCoef; ++q) (&L[0][0][0])[q * 64 + lane] = 0.f;

    // receiver recorded by this lane's axial row (first match), or -1
    int rj = -1;
    if (tr_s && i0 == 0)
        for (int r = S.nrec - 1; r >= 0; --r)
            if (own && rec_k[S.rec_off + r] == k) rj = r;
    const float srcw = k == S.src_k ? S.src_scale : 0.f;

    struct Row {
        float vr, vz, trr, ttt, tzz, trz;
    };
    // what level t keeps between two march steps
    float o_trr[T], o_ttt[T], o_tzz[T], o_trz[T], o_vz[T], n_vr[T], n_vzm[T];
    float trv[T];  // sum of the normal stresses of the axis row after each step
#pragma unroll
    for (int t = 0; t < T; ++t) {
        o_trr[t] = o_ttt[t] = o_tzz[t] = o_trz[t] = o_vz[t] = n_vr[t] = n_vzm[t] = 0.f;
        trv[t] = 0.f;
    }
    // 1/(2 r) factors of rows s, s - 1, ... (uniform: scalar registers)
    float rRs[T], rZs[T + 1], p_rR, p_rZ;
#pragma unroll
    for (int t = 0; t <= T; ++t) {
        if (t < T) rRs[t] = 0.f;
        rZs[t] = 0.f;
    }
    const int sbeg = max(0, i0 - T), send = i1 - 1 + T;
    // the row in flight: state and model of row s + 1 (at most row i1 + T <= nr)
    Row P;
    float p_lam, p_mu, p_rho;
    auto fetch = [&](int i) {
        const unsigned c = kb + (unsigned)(i * rowB), m = kb + (unsigned)(i * rowM);
        p_rR = rRt[i];
        p_rZ = rZt[i];
        P.vr = ldrow(Fi, c);
        P.vz = ldrow(Fi + cells, c);
        P.trr = ldrow(Fi + 2 * cells, c);
        P.ttt = ldrow(Fi + 3 * cells, c);
        P.tzz = ldrow(Fi + 4 * cells, c);
        P.trz = ldrow(Fi + 5 * cells, c);
        p_lam = ldrow(lam_m, m);
        p_mu = ldrow(mu_m, m);
        p_rho = ldrow(rho_m, m);
    };
    // model of the row below the first one (its coefficients only)
    float mu_prev = 0.f, rho_prev = 1.f;
    if (sbeg >= 1) {
        mu_prev = ldrow(mu_m, kb + (unsigned)((sbeg - 1) * rowM));
        rho_prev = ldrow(rho_m, kb + (unsigned)((sbeg - 1) * rowM));
    }
    fetch(sbeg);

    // One march step, straight-line over the levels.  GEN: a level may be at the
    // axis row (source and receivers), and at the levels that store the row may
    // lie outside the owned ones.  Levels that have not reached the tile yet work
    // on zeros or on rows that no later level takes.
    auto step = [&](int s, auto GENC) {
        constexpr bool GEN = decltype(GENC)::value != 0;
        Row in = P;
        // the last lane's tau_rz is halo from the first step on: its rigidity may
        // lack the neighbour
        const Coef cf = coefs(dt, p_lam, p_mu, p_rho, mu_prev, rho_prev, from_lane_above(p_mu),
                              from_lane_above(mu_prev), !GEN || s >= 1);
        mu_prev = p_mu;
        rho_prev = p_rho;
        L[(s - 1) & (kRing - 1)][4][lane] = cf.bR;  // read with row s - 1
#pragma unroll
        for (int t = T; t > 0; --t) {
            if (t < T) rRs[t] = rRs[t - 1];
            rZs[t] = rZs[t - 1];
        }
        rRs[0] = p_rR;
        rZs[0] = p_rZ;
        if (s < send) fetch(s + 1);  // uniform
        // the ring row of level t is read one level ahead
        auto ring = [&](int q) {
            const float(*Lq)[64] = L[q & (kRing - 1)];
            return Coef{Lq[0][lane], Lq[1][lane], Lq[4][lane], Lq[2][lane], Lq[3][lane]};
        };
        Coef nx = ring(s - 1);
        __builtin_amdgcn_sched_barrier(0);
        float h_vr[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int q = s - t - 1;  // takes row q + 1, finishes row q
            const Coef c = nx;
            if (t + 1 < T) {
                nx = ring(q - 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            const float rR = rRs[t], rZ = rZs[t + 1];
            // v_r at R(q + 1), v_z at Z(q)
            const float trz_km = from_lane_below(in.trz), tzz_kp = from_lane_above(o_tzz[t]);
            float Dr = fmaf(idr, in.trr - o_trr[t], (in.trz - trz_km) * idz);
            Dr = fmaf((in.trr - in.ttt) + (o_trr[t] - o_ttt[t]), rR, Dr);
            const float vr_new = fmaf(c.bR, Dr, in.vr);
            float Dr2 = fmaf(idr, in.trz - o_trz[t], (tzz_kp - o_tzz[t]) * idz);
            Dr2 = fmaf(in.trz + o_trz[t], rZ, Dr2);
            const float vz_new = fmaf(c.bZ, Dr2, o_vz[t]);
            // stresses at C(q), S(q)
            const float vz_km = from_lane_below(vz_new), vr_kp = from_lane_above(n_vr[t]);
            const float dvr = vr_new - n_vr[t], dvz = vz_new - vz_km;
            const float err = idr * dvr, ett = (vr_new + n_vr[t]) * rZ, ezz = idz * dvz;
            const float es = fmaf(idr, vz_new - n_vzm[t], (vr_kp - n_vr[t]) * idz);
            float ltr = c.cl * fmaf(idz, dvz, fmaf(idr, dvr, ett));
            if constexpr (GEN) ltr = fmaf(q == 0 ? srcw : 0.f, wv[t], ltr);
            Row out;
            out.trr = o_trr[t] + fmaf(c.c2m, err, ltr);
            out.ttt = o_ttt[t] + fmaf(c.c2m, ett, ltr);
            out.tzz = o_tzz[t] + fmaf(c.c2m, ezz, ltr);
            out.trz = fmaf(c.mS, es, o_trz[t]);
            out.vr = n_vr[t];
            out.vz = vz_new;
            o_trr[t] = in.trr;
            o_ttt[t] = in.ttt;
            o_tzz[t] = in.tzz;
            o_trz[t] = in.trz;
            o_vz[t] = in.vz;
            n_vr[t] = vr_new;
            n_vzm[t] = vz_new;
            if constexpr (GEN) trv[t] = q == 0 ? out.trr + out.ttt + out.tzz : trv[t];
            if constexpr (HIST) h_vr[t] = out.vr;
            in = out;
        }
        // row s enters the ring once its slot's last reader (row s - T) is done
        float(*Ls)[64] = L[s & (kRing - 1)];
        Ls[0][lane] = cf.cl;
        Ls[1][lane] = cf.c2m;
        Ls[2][lane] = cf.bZ;
        Ls[3][lane] = cf.mS;
        if constexpr (HIST) {  // v of row s - 1 - t after step t
            if (own) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const int q = s - 1 - t;
                    if (GEN && (q < i0 || q >= i1)) continue;  // uniform
                    float* hv = scalar_row(h_s + (long long)t * hist_stride + (long long)q * NZ);
                    strow(hv, kb, h_vr[t]);
                    strow(hv + cells_total, kb, n_vzm[t]);
                }
            }
        }
        const int q = s - T;  // the row that has left the last level
        if ((!GEN || (q >= i0 && q < i1)) && own) {
            const unsigned c = kb + (unsigned)(q * rowB);
            if (!GEN || q >= 1) {
                strow(Fo, c, in.vr);
                strow(Fo + 5 * cells, c, in.trz);
            }
            strow(Fo + cells, c, in.vz);
            strow(Fo + 2 * cells, c, in.trr);
            strow(Fo + 3 * cells, c, in.ttt);
            strow(Fo + 4 * cells, c, in.tzz);
        }
    };
    // steady steps: past the axis row at every level, on owned rows at the
    // levels that store
    const int fast0 = max(i0 + T, T + 1), fast1 = HIST ? i1 : send;
    int s = sbeg;
    while (s <= send) {
        while (s >= fast0 && s + 1 <= fast1) {  // two steps: registers swap roles
            step(s, IntC<0>{});
            step(s + 1, IntC<0>{});
            s += 2;
        }
        if (s > send) break;
        step(s, IntC<1>{});
        ++s;
    }
    if (rj >= 0)
#pragma unroll
        for (int t = 0; t < T; ++t)
            if (n0 + t < S.nt)
                tr_s[(long long)rj * S.nt + n0 + t] = trv[t] * (1.0f / 3.0f);
}

}  // namespace march
}  // namespace bhfwi
