"""The default tune: what it reports, and what a caller that names some of the
shape fields gets -- the fields left out are those of the reported tune (6x32x16
tiles, the adjoint as the forward), whatever shapes the library had chosen for
the survey."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

# one launch per block; more tiles than one launch takes; a single tall shot
SIZES = [(1, 48, 120), (12, 60, 200), (1, 320, 2048)]
DEFAULT = dict(tb_steps=6, tb_rows=32, tb_waves=16, adj_tb_steps=0, adj_tb_waves=0)


def _survey(n, nr, nz):
    import paper_2005_00281_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = workloads.tiny(nr=nr, nz=nz, nt=40)
    return P.Survey([w.shots[0]] * n, (w.NRg, w.NZg), ckpt_every=20)


def _shapes(sv):
    ks = sv.kernel_shapes()
    return ks["fwd"], ks["adj"]


@pytest.mark.parametrize("size", SIZES)
def test_partial_tunes_start_from_the_reported_default(size):
    from paper_2005_00281_amd._lib import BhfwiError
    print("[case] partial tunes", size, flush=True)
    sv = _survey(*size)
    own, t0 = _shapes(sv), sv.get_tune()
    assert {k: t0[k] for k in DEFAULT} == DEFAULT and own[0][0] >= 2
    # switches that name no shape leave the library's choice
    sv.set_tune(full_history=1, use_graph=0)
    sv.set_tune(**dict(sv.get_tune(), full_history=0))
    assert _shapes(sv) == own
    for kw, want in ((dict(tb_steps=0), (0, 0, 0)),
                     (dict(tb_steps=4), (4, 32, 16)),
                     (dict(tb_steps=6), (6, 32, 16)),
                     (dict(tb_waves=8), (6, 32, 8)),
                     (dict(tb_rows=24, tb_waves=8), (6, 24, 8)),
                     (dict(tb_steps=6, tb_rows=32, tb_waves=16), (6, 32, 16))):
        sv = _survey(*size)
        sv.set_tune(**kw)
        assert _shapes(sv) == (want, want), kw
        sv.set_tune(**t0)  # back to the library's choice
        assert _shapes(sv) == own, kw
    sv.set_tune(adj_tb_steps=1)  # the adjoint alone
    assert _shapes(sv) == ((6, 32, 16), (0, 0, 0))
    sv = _survey(*size)
    with pytest.raises(BhfwiError):  # no adjoint of that shape
        sv.set_tune(tb_steps=4, tb_rows=64, tb_waves=16)
    assert _shapes(sv) == own and sv.get_tune() == t0


def test_autotuned_shapes_are_named():
    """The autotuner's choice is reported as such, not as the default."""
    import paper_2005_00281_amd as P
    print("[case] autotune from the default tune", flush=True)
    sv = _survey(1, 24, 48)
    f = torch.ones(sv.model_shape, device=sv.device)
    lam, mu = P.moduli(3500 * f, 2000 * f, 2300 * f)
    wav = torch.zeros(sv.sizes.wavelet_elems, device=sv.device)
    t = sv.autotune(lam, mu, 2300 * f, wav, probe_steps=8)["tune"]
    assert t["adj_tb_rows"] >= 0 and sv.get_tune()["adj_tb_rows"] == t["adj_tb_rows"]
    fwd, adj = _shapes(sv)
    assert fwd[0] == (t["tb_steps"] if t["tb_steps"] >= 2 else 0)
    if t["adj_tb_steps"] >= 2:
        assert adj == (t["adj_tb_steps"], t["adj_tb_rows"], t["adj_tb_waves"])


@pytest.mark.parametrize("size,fwd", [
    # the shapes measured fastest (forward ms of 250 steps, this shape against
    # the one a count of whole columns chose)
    ((4, 50, 3000), (6, 32, 16)),   # 1.59 against 2.09 on 8x48
    ((8, 128, 512), (8, 32, 16)),   # 1.30 against 1.71 on 8x64
    ((1, 48, 6000), (6, 32, 16)),   # 0.97 against 1.10 on 8x48
    ((1, 70, 5565), (8, 48, 16)),   # 1.09 against 1.38 on 8x64
    ((1, 176, 3391), (6, 32, 16)),  # 1.15 against 1.38 on 8x64
    ((10, 148, 267), (8, 32, 16)),  # 1.30 against 1.65 on 8x64
    ((10, 50, 720), (8, 64, 16)),   # 1.41 against 1.52 on 6x32: thin, in PML tiles only
    ((1, 128, 512), (8, 32, 16)),   # one launch per block
    ((8, 256, 4096), (8, 48, 16))])  # beside the marches
def test_own_forward_shape(size, fwd):
    import paper_2005_00281_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the shapes were measured on 256 compute units")
    print("[case] own shape", size, flush=True)
    n, nr, nz = size
    one = workloads.tiny(nr=24, nz=48, nt=40).shots[0]
    sh = workloads.Shot(nr, nz, 20, 20, one.dr, one.dz, one.dt, 40, one.f0, one.vmax, 25,
                        one.rec_k, one.wavelet)
    sv = P.Survey([sh] * n, (nr + 20, nz + 40), ckpt_every=20)
    assert _shapes(sv) == (fwd, (6, 32, 16))
