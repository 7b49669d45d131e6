"""The register marches that run the PML-free tiles of surveys with enough
columns: parity with the oracle at the edges of their tiles (several radial
tiles per column, tiles at the axis, remainders of the time blocks, ragged
records that end inside a block, receivers and sources on the axis row)."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from util import geom, rel_l2

pytestmark = pytest.mark.gpu


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def _f32(a):
    return torch.as_tensor(np.ascontiguousarray(a, np.float32), device=_dev())


def _batch(nshot, nr, nz, pml, nt):
    """nshot shots over one small model, enough of them that the marches run:
    windows shifted by one axial row, two record lengths."""
    w = workloads.tiny(nr=nr, nz=nz + nshot - 1, p=pml, nt=nt)
    one = workloads.tiny(nr=nr, nz=nz, p=pml, nt=nt).shots[0]
    shots = []
    for s in range(nshot):
        n = nt if s % 3 else nt - 3  # records that end inside a block
        shots.append(workloads.Shot(one.nr, one.nz, one.pr, one.pz, one.dr, one.dz, one.dt, n,
                                    one.f0, w.shots[0].vmax, one.src_k, one.rec_k,
                                    one.wavelet[:n], s))
    w.shots = shots
    return w


@pytest.mark.parametrize("tb,atb,nt,K", [(8, 6, 301, 100), (6, 8, 277, 95), (4, 4, 270, 63)])
@pytest.mark.parametrize("extra", ["", "ex", "wavelet"])
def test_marches_match_the_oracle(tb, atb, nt, K, extra):
    """300 shots of 156 x 300 cells: four clear columns each, cut into two radial
    tiles that the marches run.  Traces of three shots and, with residuals on
    those shots only, the gradient (the rows around the cut also on their own)
    and the optional outputs against the oracle; bars as everywhere: 1e-4
    traces, 1e-3 gradients, 1e-4 illumination and pseudo-Hessian."""
    import paper_2005_00281_amd as P
    print("[case] marches", tb, atb, nt, K, extra, flush=True)
    w = _batch(300, 150, 288, 6, nt)
    sv = P.Survey(w.shots, (w.NRg, w.NZg), ckpt_every=K)
    sv.set_tune(tb_steps=tb, tb_rows=48, tb_waves=16, adj_tb_steps=atb, adj_tb_rows=32,
                adj_tb_waves=16)
    rho = _f32(w.rho)
    lam, mu = P.moduli(_f32(w.vp_start), _f32(w.vs_start), rho)
    wav = sv.pack_wavelets([s.wavelet for s in w.shots])
    tr = sv.unpack_traces(sv.fwd_model(lam, mu, rho, wav, store_ckpt=True))
    pick = (0, 149, 299)
    rng = np.random.default_rng(5)
    r = np.zeros(sv.sizes.trace_elems, np.float32)
    g_o = None
    for s in pick:
        sh = w.shots[s]
        lo, mo = oracle.moduli(w.window(w.vp_start, s), w.window(w.vs_start, s),
                               np.ascontiguousarray(w.window(w.rho, s)))
        ro = np.ascontiguousarray(w.window(w.rho, s))
        d = oracle.forward(geom(sh), lo, mo, ro, sh.wavelet)
        assert rel_l2(tr[s], d) <= 1e-4
        res = rng.standard_normal(d.shape)
        off = sv.trace_slices()[s][0]
        r[off: off + res.size] = res.ravel()
        out = oracle.gradient(geom(sh), lo, mo, ro, sh.wavelet, res, seg=20,
                              density=extra == "ex", hessian=extra == "ex")
        g_o = g_o or []
        g_o.append((s, sh, out))
    if extra == "ex":
        acc, acc_r, acc_h = sv.adjoint_model_ex(lam, mu, rho, wav, _f32(r), density=True,
                                                hessian=True)
        gr = sv.gradient_density(rho, acc_r).cpu().numpy()
    elif extra == "wavelet":
        acc, gw = sv.adjoint_model_wavelet(lam, mu, rho, wav, _f32(r))
    else:
        acc = sv.adjoint_model(lam, mu, rho, wav, _f32(r))
    gl, gm, _ = (t.cpu().numpy() for t in sv.gradient(mu, acc))
    views = sv.acc_views(acc)
    want_l, want_m, want_r = np.zeros_like(gl), np.zeros_like(gm), np.zeros_like(gm)
    for s, sh, out in g_o:
        win = (slice(0, sh.NR), slice(s, s + sh.NZ))
        want_l[win] += out[0]
        want_m[win] += out[1]
        assert rel_l2(views[s][3].cpu().numpy(), out[2]) <= 1e-4
        if extra == "ex":
            want_r[win] += out[3]
    assert rel_l2(gl, want_l) <= 1e-3 and rel_l2(gm, want_m) <= 1e-3
    for cut in (slice(55, 90), slice(130, 156)):
        assert rel_l2(gl[cut], want_l[cut]) <= 1e-3 and rel_l2(gm[cut], want_m[cut]) <= 1e-3
    if extra == "ex":
        assert rel_l2(gr, want_r) <= 1e-3
        s, sh, out = g_o[1]
        hv = torch.stack([acc_h[:sv.sizes.cells], acc_h[sv.sizes.cells:]])
        base = sum((x.NR * x.NZ + 63) // 64 * 64 for x in w.shots[:s])
        for q in range(2):
            h = hv[q][base: base + sh.cells].view(sh.NR, sh.NZ).cpu().numpy()
            assert rel_l2(h, out[4 + q]) <= 1e-4
    if extra == "wavelet":
        # <F w, r> = <w, F^T r> per shot: the wavelet gradient against the traces
        o, gwn = 0, gw.cpu().numpy().astype(np.float64)
        for s, sh in enumerate(w.shots):
            if s in pick:
                off, nrec, n = sv.trace_slices()[s]
                lhs = float(np.dot(tr[s].ravel().astype(np.float64),
                                   r[off: off + nrec * n].astype(np.float64)))
                rhs = float(np.dot(gwn[o: o + n], sh.wavelet.astype(np.float32)))
                scale = np.linalg.norm(tr[s].astype(np.float64)) * np.linalg.norm(
                    r[off: off + nrec * n])
                assert abs(lhs - rhs) <= 1e-5 * scale
            o += sh.nt


@pytest.mark.parametrize("T", [4, 6])
def test_last_owned_lane(T):
    """Column by column, the march's correlations against those of the same shot
    alone, which the LDS tiles run: the lane beside a strip's last sound one must
    not reach it within a block.  Bar: the two differ by the rounding of some 300
    steps, about 6e-8 * sqrt(4 * 300) = 2e-6, times 5 for one column's norm."""
    import paper_2005_00281_amd as P
    print("[case] march strips", T, flush=True)
    w = _batch(300, 150, 288, 6, 301)
    rng = np.random.default_rng(6)
    rho = _f32(w.rho)
    lam, mu = P.moduli(_f32(w.vp_start), _f32(w.vs_start), rho)
    acc, s = [], 149
    for shots in (w.shots, w.shots[s:s + 1]):
        sv = P.Survey(shots, (w.NRg, w.NZg), ckpt_every=50)
        sv.set_tune(tb_steps=8, tb_rows=48, tb_waves=16, adj_tb_steps=T, adj_tb_rows=32,
                    adj_tb_waves=16)
        sv.fwd_model(lam, mu, rho, sv.pack_wavelets([x.wavelet for x in shots]),
                     store_ckpt=True)
        r = np.zeros(sv.sizes.trace_elems, np.float32)
        j = len(acc) == 0 and s or 0
        off, nrec, n = sv.trace_slices()[j]
        if not acc:
            res = rng.standard_normal(nrec * n).astype(np.float32)
        r[off: off + nrec * n] = res
        a = sv.adjoint_model(lam, mu, rho, sv.pack_wavelets([x.wavelet for x in shots]), _f32(r))
        acc.append([v.cpu().numpy().astype(np.float64) for v in sv.acc_views(a)[j]])
    for q, (a, b) in enumerate(zip(*acc)):
        e, n = np.linalg.norm(a - b, axis=0), np.linalg.norm(b, axis=0)
        assert (e <= 1e-5 * np.maximum(n, n.mean())).all(), (q, (e / np.maximum(n, n.mean())).max())
