"""Pair densities of many k-points (grids and pair kernels launched for groups
of k-points) against the same k-points one call at a time: the same values
bit for bit, on grids of each kind, with a last group that is not full."""

import numpy as np
import pytest

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


# lane kernels with groups of 32 (36 k-points), the generic pair kernel, the
# umklapp in every direction, and planes too large for LDS (72^2 in FP64)
@pytest.mark.parametrize("edge, kmesh, iq, gpsi, ng, prec", [
    (16, (4, 3, 3), (1, 2, 0), 3.2, 33, 0), (16, (4, 3, 3), (3, 1, 2), 3.2, 33, 1), (27, (2, 2, 2), (1, 1, 1), 6.0, 300, 0),
    (20, (5, 1, 1), (2, 0, 0), 3.0, 100, 2), (72, (2, 1, 1), (1, 0, 0), 30.0, 27, 0)])
def test_groups_equal_single_k_points(ctx, rp, edge, kmesh, iq, gpsi, ng, prec):
    from paper_2001_02351_amd import path
    from synth import make_problem
    a = 2.0 * np.pi
    p = make_problem(name="kgroup", a_bohr=a, fft=(edge,) * 3, kmesh=kmesh, iq=iq, nocc=2, nemp=3, gpsi=gpsi, ng=ng,
                     freq_eV=[0.0], delta_eV=0.1, seed=edge)
    d = path.DeviceInputs(p)
    print(f"[kgroup] edge={edge} nk={d.nk} grid={rp.rp_pair_grid(d.cell, p.iq, d.mmax, p.gsph, prec)}", flush=True)
    M = path.pair_density(ctx, d, 0, d.nk, prec=prec)
    rp.rp_synchronize(ctx)
    assert bool(torch.isfinite(M).all()) and float(M.abs().max()) > 0
    for k in range(d.nk):
        one = path.pair_density(ctx, d, k, k + 1, prec=prec)
        rp.rp_synchronize(ctx)
        assert torch.equal(M[6 * k:6 * k + 6], one)
