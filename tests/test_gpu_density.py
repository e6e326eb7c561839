"""Direct and exchange densities and their quadratic forms where the kernels'
routes change: grids of the lane kernel and others, lists whose m3 window
wraps around the axis, one to several vectors per thread, few densities (their
planes shared by workgroups) and many, more than 16 orbitals, and lists of R
that hold twins (R, i, j) and (-R, j, i), some of them at half-cell
boundaries.  The orbitals are random on the grid, so that every image and cut
counts.  Against the oracle, 1e-10 of the largest value as elsewhere.
"""

import numpy as np
import pytest

from oracle import qsum

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_02351_amd as rp
    rp.load()
    return rp


@pytest.fixture(scope="module")
def ctx(rp):
    c = rp.Context(0)
    yield c
    c.close()


def _dev(a):
    a = np.ascontiguousarray(a)
    return torch.from_numpy(a.view(np.float64).reshape(a.shape + (2,)) if a.dtype == np.complex128 else a).cuda()


SYM = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, -1), (0, -1, 1), (1, 0, 0)]
WIDE = [(i, j, k) for i in (0, 1, 2) for j in (-1, 0, 1) for k in (0, 1, 2, 3)]


@pytest.mark.parametrize("fft, iq, nwan, cells, ng, ntail, nfreq", [
    ((16, 16, 16), (1, 0, 2), 3, SYM, 33, 40, 2), ((12, 16, 16), (0, 0, 0), 3, SYM, 70, 0, 1),
    ((20, 20, 20), (0, 1, 0), 2, SYM, 1, 7, 3), ((18, 18, 18), (1, 1, 1), 3, SYM, 65, 10, 2),
    ((9, 24, 24), (2, 1, 0), 3, WIDE, 100, 1000, 1), ((16, 16, 16), (1, 2, 2), 2, SYM, 31, 2600, 1),
    ((16, 16, 16), (0, 2, 1), 17, SYM[:3], 64, 5, 1), ((16, 16, 16), (0, 0, 0), 4, WIDE, 48, 4800, 1)])
@pytest.mark.parametrize("special", [False, True])
def test_densities_and_quadratic_forms(rp, ctx, fft, iq, nwan, cells, ng, ntail, nfreq, special):
    print(f"[density] fft={fft} iq={iq} nwan={nwan} nR={len(cells)} ng={ng} ntail={ntail} special={special}", flush=True)
    rng = np.random.default_rng([fft[0], nwan, ng])
    kmesh, lat = (3, 4, 3), np.diag([7.0, 8.0, 9.0])
    # special centres put grid points on half-cell boundaries, exactly or up to rounding
    cen = rng.choice([0.0, 0.5, 0.25, 1.0 / 3.0, 2.0 / 3.0], (nwan, 3)) if special else rng.uniform(0, 1, (nwan, 3))
    phi = rng.standard_normal((nwan,) + fft)
    R = np.array(cells, np.int32)
    s = np.arange(-8, 9)
    allg = np.stack(np.meshgrid(s, s, s, indexing="ij"), -1).reshape(-1, 3)
    gl = allg[np.argsort(qsum.qg_norm(lat, kmesh, iq, allg), kind="stable")][:ng + ntail].astype(np.int32)
    E = np.eye(ng)[None] + 0.1 * (rng.standard_normal((nfreq, ng, ng)) + 1j * rng.standard_normal((nfreq, ng, ng)))
    gamma = not any(iq)
    n_u = np.stack([qsum.exchange_ntilde(lat, fft, kmesh, iq, phi[i:i + 1], cen[i:i + 1], [[0, 0, 0]], gl)[0, 0, 0]
                    for i in range(nwan)])
    n_x = qsum.exchange_ntilde(lat, fft, kmesh, iq, phi, cen, R, gl)
    want = qsum.qterm(lat, kmesh, iq, n_u, n_x, ng, E, R, gl,
                      head_avg=qsum.cell_average(lat, kmesh) if gamma else None)
    cell = rp.make_cell(lat, fft, kmesh)
    out = {k: torch.full(want[k].shape + (2,), float("nan"), dtype=torch.float64, device="cuda") for k in "UJVX"}
    rp.rp_wannier_qterm(ctx, cell, iq, nwan, _dev(phi), cen, R, ng, gl[:ng], ntail, gl[ng:], nfreq, _dev(E), 0, **out)
    rp.rp_synchronize(ctx)
    for k in "UJVX":
        got = out[k].cpu().numpy()
        got = got[..., 0] + 1j * got[..., 1]
        assert np.abs(got - want[k]).max() <= 1e-10 * np.abs(want[k]).max(), k
    if not gamma:   # the same sums without R, through the projection entry point
        W = torch.full((nfreq, nwan, nwan, 2), float("nan"), dtype=torch.float64, device="cuda")
        rp.rp_wannier_W(ctx, cell, iq, nwan, _dev(phi), cen, ng, gl[:ng], ntail, gl[ng:], nfreq, _dev(E), W)
        rp.rp_synchronize(ctx)
        got = torch.view_as_complex(W).cpu().numpy()
        assert np.abs(got - want["U"][:, cells.index((0, 0, 0))]).max() <= 1e-10 * np.abs(want["U"]).max()


def test_batch_graphs_survive_a_q_term(rp, ctx):
    """A repeated batch relaunches its graphs: a q-term in between leaves what they read alone."""
    from paper_2001_02351_amd import path
    from synth import make_problem
    p = make_problem(name="keep", a_bohr=6.0, fft=(16,) * 3, kmesh=(2, 2, 2), iq=(1, 0, 0), nocc=2, nemp=3, gpsi=3.5,
                     ng=30, freq_eV=[0.0, 3.0], delta_eV=0.1, nwan=3, seed=4)
    d = path.DeviceInputs(p)
    first = [c.clone() for c in path.chi0_batch(ctx, [d], prec=0)]
    chis = path.chi0_batch(ctx, [d], prec=0)
    probs = [path.batch_problem(d, chis[0])]
    rp.rp_chi0_batch(ctx, probs, 0)
    E = torch.zeros(2, 30, 30, 2, dtype=torch.float64, device="cuda")
    X = torch.zeros(125, 3, 3, 2, dtype=torch.float64, device="cuda")
    R = np.array([(i, j, k) for i in range(5) for j in range(5) for k in range(5)], np.int32)
    rp.rp_wannier_qterm(ctx, d.cell, p.iq, 3, d.phi, p.centre_frac, R, 30, p.gsph, 0, None, 2, E, 0, X=X)
    chis[0].fill_(float("nan"))
    rp.rp_chi0_batch(ctx, probs, 0)
    rp.rp_synchronize(ctx)
    assert torch.equal(chis[0], first[0])
