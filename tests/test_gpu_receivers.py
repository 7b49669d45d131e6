"""Receivers of the time-blocked kernels: they are staged 64 at a time, so more
than 64 of them, receivers on every axial row (tile edges and both PML layers
included) and in any order give the oracle's traces and gradient."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from util import geom, rel_l2

pytestmark = pytest.mark.gpu


def _f32(a):
    return torch.as_tensor(np.ascontiguousarray(a, np.float32), device="cuda:0")


@pytest.mark.parametrize("nrec", [1, 64, 65, 162])
@pytest.mark.parametrize("T", [4, 6, 8])
def test_many_receivers(nrec, T):
    """One shot of 156 x 162 cells in 32-row tiles; the receivers are a shuffled
    subset of the axial rows.  Bars as everywhere: 1e-4 traces, 1e-3 gradient."""
    import paper_2005_00281_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] receivers", nrec, T, flush=True)
    w = workloads.tiny(nr=150, nz=150, p=6, nt=203)
    one = w.shots[0]
    rng = np.random.default_rng(nrec)
    rec = [int(k) for k in rng.permutation(one.NZ)[:nrec]]
    sh = workloads.Shot(one.nr, one.nz, one.pr, one.pz, one.dr, one.dz, one.dt, one.nt, one.f0,
                        one.vmax, one.src_k, rec, one.wavelet, 0)
    sv = P.Survey([sh], (w.NRg, w.NZg), ckpt_every=50)
    sv.set_tune(tb_steps=T, tb_rows=32, tb_waves=16, adj_tb_steps=T, adj_tb_rows=32,
                adj_tb_waves=16)
    rho = _f32(w.rho)
    lam, mu = P.moduli(_f32(w.vp_start), _f32(w.vs_start), rho)
    wav = sv.pack_wavelets([sh.wavelet])
    tr = sv.unpack_traces(sv.fwd_model(lam, mu, rho, wav, store_ckpt=True))[0]
    lo, mo = oracle.moduli(w.vp_start, w.vs_start, w.rho)
    d = oracle.forward(geom(sh), lo, mo, w.rho, sh.wavelet)
    assert rel_l2(tr, d) <= 1e-4
    res = rng.standard_normal(d.shape)
    out = oracle.gradient(geom(sh), lo, mo, w.rho, sh.wavelet, res, seg=20)
    acc = sv.adjoint_model(lam, mu, rho, wav, _f32(res.ravel()))
    gl, gm, _ = (t.cpu().numpy() for t in sv.gradient(mu, acc))
    assert rel_l2(gl, out[0]) <= 1e-3 and rel_l2(gm, out[1]) <= 1e-3
