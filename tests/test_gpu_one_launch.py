"""Blocks of surveys whose tiles fit the GPU in one round, run in one launch:
parity with the oracle on two shots of different size and record length."""
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


@pytest.mark.parametrize("order", [2, 4])
def test_one_launch_blocks_match_the_oracle(order):
    """A survey whose interior and PML tiles run in one launch per block: two
    shots of different size and record length, default tune."""
    import paper_2005_00281_amd as P
    print("[case] one-launch blocks, order", order, flush=True)
    w = workloads.batched_uneven(nshot=2, h=5e-3, p=8, nrec=3, nz_choices=(160, 230),
                                 nr_choices=(70, 90), f0_range=(15e3, 20e3), rec_ms=(0.2, 0.3))
    sv = P.Survey(w.shots, (w.NRg, w.NZg), ckpt_every=40, order=order)
    rho = _f32(w.rho)
    lam, mu = P.moduli(_f32(w.vp_start), _f32(w.vs_start), rho)
    wav = sv.pack_wavelets([s.wavelet for s in w.shots])
    tr = sv.unpack_traces(sv.fwd_model(lam, mu, rho, wav, store_ckpt=True))
    rng = np.random.default_rng(6)
    r, want = [], (np.zeros(w.rho.shape), np.zeros(w.rho.shape))
    kw = {} if order == 2 else dict(order=4)
    for s, sh in enumerate(w.shots):
        ro = np.ascontiguousarray(w.window(w.rho, s))
        lo, mo = oracle.moduli(w.window(w.vp_start, s), w.window(w.vs_start, s), ro)
        d = oracle.forward(geom(sh), lo, mo, ro, sh.wavelet, **kw)
        assert rel_l2(tr[s], d) <= 1e-4
        res = rng.standard_normal(d.shape)
        r.append(res.ravel())
        out = oracle.gradient(geom(sh), lo, mo, ro, sh.wavelet, res, **kw)
        win = (slice(0, sh.NR), slice(sh.win_k0, sh.win_k0 + sh.NZ))
        want[0][win] += out[0]
        want[1][win] += out[1]
    acc = sv.adjoint_model(lam, mu, rho, wav, _f32(np.concatenate(r)))
    gl, gm, _ = (t.cpu().numpy() for t in sv.gradient(mu, acc))
    assert rel_l2(gl, want[0]) <= 1e-3 and rel_l2(gm, want[1]) <= 1e-3
