"""Which form the temporally blocked launches run -- register marches, LDS tiles
clear of the PML beside PML tiles, or one PML launch per block -- asserted
through bhfwi_kernel_tiles, and each form against the oracle where its tiles
meet.  Bars as everywhere: 1e-4 traces and illumination, 1e-3 gradients, 1e-4
pseudo-Hessian."""
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


def _batch(sizes, nt, pml=6, pr=None):
    """Shots of the given (nr, nz) over one small model, windows shifted by one
    axial row each; every third record ends inside a time block.  pr: rows of
    the radial layer where they are not those of the axial layers."""
    pr = pml if pr is None else pr
    nr, nz = max(r for r, _ in sizes), max(z + s for s, (_, z) in enumerate(sizes))
    w = workloads.tiny(nr=nr, nz=nz, p=pml, nt=nt, dt=0.75e-6)
    shots = []
    for s, (r, z) in enumerate(sizes):
        one = workloads.tiny(nr=r, nz=z, p=pml, nt=nt, dt=0.75e-6).shots[0]
        n = nt if s % 3 else nt - 3
        shots.append(workloads.Shot(r, z, pr, pml, one.dr, one.dz, one.dt, n, one.f0,
                                    w.shots[0].vmax, one.src_k, one.rec_k, one.wavelet[:n], s))
    w.shots = shots
    return w


class _Check:
    """Survey of a batch in a tune, with residuals on the picked shots, and the
    oracle's traces and gradients of those."""

    def __init__(self, w, pick, K=50):
        self.w, self.pick, self.K = w, pick, K
        rng = np.random.default_rng(5)
        self.d, self.res, self.out = {}, {}, {}
        for s in pick:
            sh, ro = w.shots[s], np.ascontiguousarray(w.window(w.rho, s))
            lo, mo = oracle.moduli(w.window(w.vp_start, s), w.window(w.vs_start, s), ro)
            self.d[s] = oracle.forward(geom(sh), lo, mo, ro, sh.wavelet)
            self.res[s] = rng.standard_normal(self.d[s].shape)
            self.out[s] = oracle.gradient(geom(sh), lo, mo, ro, sh.wavelet, self.res[s], seg=20,
                                          density=True, hessian=True)
        self.want = [np.zeros(w.rho.shape) for _ in range(3)]
        for s in pick:
            sh = w.shots[s]
            win = (slice(0, sh.NR), slice(s, s + sh.NZ))
            for q, j in enumerate((0, 1, 3)):
                self.want[q][win] += self.out[s][j]

    def survey(self, **tune):
        import paper_2005_00281_amd as P
        w = self.w
        self.sv = sv = P.Survey(w.shots, (w.NRg, w.NZg), ckpt_every=self.K)
        sv.set_tune(**tune)
        self.rho = _f32(w.rho)
        self.lam, self.mu = P.moduli(_f32(w.vp_start), _f32(w.vs_start), self.rho)
        self.wav = sv.pack_wavelets([x.wavelet for x in w.shots])
        return sv

    def run(self, bands=()):
        """Traces, then the gradient without and with the extra outputs; the
        rows of `bands` also on their own."""
        sv, w = self.sv, self.w
        args = (self.lam, self.mu, self.rho, self.wav)
        tr = sv.unpack_traces(sv.fwd_model(*args, store_ckpt=True))
        r = np.zeros(sv.sizes.trace_elems, np.float32)
        for s in self.pick:
            assert rel_l2(tr[s], self.d[s]) <= 1e-4, s
            off = sv.trace_slices()[s][0]
            r[off: off + self.res[s].size] = self.res[s].ravel()
        base = np.cumsum([0] + [(x.cells + 63) // 64 * 64 for x in w.shots])
        for extra in (False, True):
            acc, acc_r, acc_h = sv.adjoint_model_ex(*args, _f32(r), density=extra, hessian=extra)
            g = list(sv.gradient(self.mu, acc)[:2])
            if extra:
                g.append(sv.gradient_density(self.rho, acc_r))
            for a, b in zip(g, self.want):
                a = a.cpu().numpy()
                for band in (slice(0, None),) + tuple(bands):
                    assert rel_l2(a[band], b[band]) <= 1e-3, (extra, band)
            views = sv.acc_views(acc)
            for s in self.pick:
                sh = w.shots[s]
                il = views[s][3].cpu().numpy()
                for band in (slice(0, None),) + tuple(bands):
                    assert rel_l2(il[band], self.out[s][2][band]) <= 1e-4, (extra, s, band)
                for q in range(2 if extra else 0):
                    h = acc_h[q * sv.sizes.cells + base[s]:][:sh.cells]
                    h = h.view(sh.NR, sh.NZ).cpu().numpy()
                    for band in (slice(0, None),) + tuple(bands):
                        assert rel_l2(h[band], self.out[s][4 + q][band]) <= 1e-4, (s, q, band)


@pytest.mark.parametrize("T", [4, 6])
def test_rows_beside_the_cuts_of_the_marches(T):
    """300 shots of 156 x 300 cells run the marches in both directions; the T
    rows on either side of every cut between two march tiles, and of the cut
    between the last one and the LDS tiles of the radial layer, on their own.
    The record holds the way to the outermost rows and back: 2 x 150 cells at
    some 0.52 cells (3500 m/s) per step, 572 steps."""
    print("[case] march cuts", T, flush=True)
    c = _Check(_batch([(150, 288)] * 300, 640), (0, 149))
    sv = c.survey(tb_steps=8, tb_rows=48, tb_waves=16, adj_tb_steps=T, adj_tb_rows=32,
                  adj_tb_waves=16)
    bands = []
    for part, t in (("fwd", 8), ("adj_x", T)):
        R, clear, pml = sv.kernel_tiles()[part]
        top = 150 - t
        assert R >= 64 and pml > 0
        n = -(-top // R)
        assert n >= 2 and clear % (300 * n) == 0
        bands += [slice(cut - t, cut + t) for cut in [top * j // n for j in range(1, n + 1)]]
    c.run(bands)


MID = dict(tb_steps=8, tb_rows=48, tb_waves=16, adj_tb_steps=6, adj_tb_rows=32, adj_tb_waves=16)


@pytest.mark.parametrize("overlap", [0, 1])
def test_lds_tiles_between_one_launch_and_the_marches(overlap):
    """12 shots of 126 x 252 cells: more tiles than one launch per block takes
    and too few columns for the marches, so the PML-free LDS kernels run (with
    overlap, one more forward tile per clear column)."""
    print("[case] LDS tiles, overlap", overlap, flush=True)
    c = _Check(_batch([(120, 240)] * 12, 200), (0, 7))
    sv = c.survey(fwd_tile_overlap=overlap, **MID)
    tiles = sv.kernel_tiles()
    # 3 clear columns of 48: tiles at rows 0, 32, 64 and, overlapping, at 80
    assert tiles["fwd"][:2] == (0, 12 * 3 * (4 if overlap else 3))
    for part in ("adj", "adj_x"):
        assert tiles[part][0] == 0 and tiles[part][1] > 0 and tiles[part][2] > 0
    c.run()
    if not overlap:  # the wavelet record's kernel: <F w, r> = <w, F^T r>
        tr = sv.unpack_traces(sv.fwd_model(c.lam, c.mu, c.rho, c.wav, store_ckpt=True))
        r = np.random.default_rng(2).standard_normal(sv.sizes.trace_elems).astype(np.float32)
        _, gw = sv.adjoint_model_wavelet(c.lam, c.mu, c.rho, c.wav, _f32(r))
        gw, o = gw.cpu().numpy().astype(np.float64), 0
        for (off, nrec, n), x, t in zip(sv.trace_slices(), c.w.shots, tr):
            rs = r[off: off + nrec * n].astype(np.float64)
            lhs = float(np.dot(t.ravel().astype(np.float64), rs))
            rhs = float(np.dot(gw[o: o + n], x.wavelet.astype(np.float32)))
            assert abs(lhs - rhs) <= 1e-5 * np.linalg.norm(t.astype(np.float64)) * \
                np.linalg.norm(rs)
            o += n


@pytest.mark.parametrize("mode", [dict(rec_overlap=1), dict(full_history=1), dict(pml_overlap=1)])
def test_marches_with_odd_shots_and_history_modes(mode):
    """Among 300 marched shots one whose interior is thinner than a time block
    (nr = 5) and one without a column clear of the axial layers (nz = 40): they
    run in PML tiles only.  With the recompute overlapped (marches and PML tiles
    of a block in one stream), the whole history, and the PML stream asked for."""
    print("[case] marches", mode, flush=True)
    sizes = [(150, 288)] * 300
    sizes[10], sizes[20] = (5, 288), (150, 40)
    c = _Check(_batch(sizes, 200), (10, 20, 299))
    sv = c.survey(**dict(MID, **mode))
    tiles = sv.kernel_tiles()
    assert tiles["fwd"][0] >= 64 and tiles["adj"][0] >= 64
    c.run()


def test_one_launch_and_one_step_report_their_tiles():
    print("[case] tile report", flush=True)
    c = _Check(_batch([(60, 200)], 40), ())
    sv = c.survey(**MID)
    for part in ("fwd", "adj"):  # every tile in the PML kernel
        assert sv.kernel_tiles()[part][:2] == (0, 0) and sv.kernel_tiles()[part][2] > 0
    sv.set_tune(tb_steps=0, adj_tb_steps=1)
    assert set(sv.kernel_tiles().values()) == {(0, 0, 0)}


@pytest.mark.parametrize("rows", [32, 48, 64])
def test_eight_step_adjoints_keep_their_lds_tiles(rows):
    """An adjoint of eight steps per launch has no march (it would spill): a
    survey whose forward marches runs it on the LDS tiles of its shape."""
    print("[case] eight-step adjoint, rows", rows, flush=True)
    c = _Check(_batch([(150, 288)] * 300, 200), (0, 299))
    sv = c.survey(**dict(MID, adj_tb_steps=8, adj_tb_rows=rows))
    tiles = sv.kernel_tiles()
    assert tiles["fwd"][0] >= 64
    for part in ("adj", "adj_x"):
        assert tiles[part][0] == 0 and tiles[part][1] > 0 and tiles[part][2] > 0
    c.run()


@pytest.mark.parametrize("pml", [6, 0])
def test_marches_without_a_radial_layer(pml):
    """Without a radial layer the march's last row is the grid's: what the last
    step of a column fetches ahead must stay on it.  With and without axial
    layers; the record holds the way to that row and back."""
    print("[case] marches, no radial layer, axial", pml, flush=True)
    c = _Check(_batch([(150, 288)] * 300, 640, pml=pml, pr=0), (0, 299))
    sv = c.survey(**MID)
    tiles = sv.kernel_tiles()
    assert tiles["fwd"][0] >= 64 and tiles["adj"][0] >= 64
    c.run([slice(138, 150)])


def test_order4_reports_the_tiles_of_its_blocks():
    import paper_2005_00281_amd as P
    print("[case] tile report, order 4", flush=True)
    _dev()
    w = workloads.tiny(nr=60, nz=200, nt=40)
    sv = P.Survey(w.shots, (w.NRg, w.NZg), ckpt_every=20, order=4)
    assert {(m, a) for m, a, _ in sv.kernel_tiles().values()} == {(0, 0)}  # one launch
    assert sv.kernel_tiles()["adj"][2] > 0
    sv.set_order4_blocks(0)
    assert set(sv.kernel_tiles().values()) == {(0, 0, 0)}


def test_graph_replays_of_the_marches_equal_eager_launches():
    """The captured sequence of marches beside PML tiles on the forked stream,
    replayed with eager work and synchronisations in between, gives the eager
    launches' traces and accumulators bit for bit."""
    print("[case] march graph replays", flush=True)
    c = _Check(_batch([(150, 288)] * 300, 100), ())
    out = {}
    for graph in (0, 1):
        sv = c.survey(use_graph=graph, **MID)
        assert sv.kernel_tiles()["fwd"][0] >= 64 and sv.kernel_tiles()["adj"][0] >= 64
        args = (c.lam, c.mu, c.rho, c.wav)
        r = torch.randn(sv.sizes.trace_elems, device=sv.device,
                        generator=torch.Generator(device=sv.device).manual_seed(4))
        tr = torch.empty_like(r)
        acc = torch.empty(sv.sizes.acc_elems, device=sv.device)
        for rep in range(4 if graph else 1):
            tr.fill_(float("nan"))
            acc.fill_(float("nan"))
            sv.fwd_model(*args, store_ckpt=True, traces=tr)
            sv.adjoint_model(*args, r, acc=acc)
            torch.cuda.synchronize()
            assert (c.lam * 2).sum().item() > 0  # unrelated eager work between replays
            views = [v.clone() for v in sv.acc_views(acc)]
            if not graph:
                out["tr"], out["acc"] = tr.clone(), views
            else:
                assert torch.equal(tr, out["tr"]), rep
                assert all(torch.equal(a, b) for a, b in zip(views, out["acc"])), rep
