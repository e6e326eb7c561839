"""The tetrahedron weights where their evaluation changes: frequencies far
from a pair's energies (moment series), near them (divided differences), both
in one workgroup; flat and nearly flat bands; pair and frequency counts around
the workgroup's 32 and 16; the Fermi level through some of a pair's
tetrahedra.  Against the oracle to 1e-12 of the largest weight, the bar of
the weights elsewhere (1e-11 where tetrahedra are cut).
"""

import numpy as np
import pytest

import oracle
from oracle import metal

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


def _weights(rp, ctx, kmesh, iq, E, T, o, e, k1, freq, delta, mode):
    cell = rp.make_cell(np.eye(3) * 7.0, (8, 8, 8), kmesh)
    w = torch.full((len(freq), k1 * (e[1] - e[0]) * (o[1] - o[0]), 2), float("nan"), dtype=torch.float64, device="cuda")
    Ed = torch.from_numpy(np.ascontiguousarray(E)).cuda()
    Td = None if T is None else torch.from_numpy(T).cuda()
    rp.rp_weights(ctx, cell, iq, E.shape[1], Ed, Td, *o, *e, 0, k1, len(freq), freq, delta, mode, w)
    rp.rp_synchronize(ctx)
    a = w.cpu().numpy()
    return a[..., 0] + 1j * a[..., 1]


# spread: 0 flat bands, 1e-9 nearly flat, 0.3 mostly series, 3 mostly divided differences
@pytest.mark.parametrize("spread", [0.0, 1e-9, 0.3, 3.0])
@pytest.mark.parametrize("nocc, nemp, k1, nfreq", [(1, 1, 1, 1), (1, 31, 1, 17), (3, 11, 1, 2), (4, 8, 3, 33)])
@pytest.mark.parametrize("imag", [False, True])
def test_weights_near_and_far(rp, ctx, spread, nocc, nemp, k1, nfreq, imag):
    print(f"[weights] spread={spread} pairs={nocc * nemp * k1} nfreq={nfreq} imag={imag}", flush=True)
    kmesh, iq = (3, 2, 2), (1, 0, 1)
    rng = np.random.default_rng([nocc, nemp, nfreq])
    centre = np.concatenate([np.sort(rng.uniform(-8, -4, nocc)), np.sort(rng.uniform(4, 16, nemp))])
    E = centre + spread * rng.uniform(-1, 1, (12, nocc + nemp))
    T = np.zeros_like(E)
    T[:, nocc - 1:nocc + 1] = rng.uniform(0, 1, (12, 2))
    freq = 1j * np.linspace(0.0, 40.0, nfreq) if imag else np.linspace(0.0, 24.0, nfreq) + 0j
    delta = 0.0 if imag else 0.1
    got = _weights(rp, ctx, kmesh, iq, E, T, (0, nocc), (nocc, nocc + nemp), k1, freq, delta, rp.RP_W_TETRA)
    want = oracle.weights(kmesh, iq, E, T, 0, nocc, nocc, nocc + nemp, 0, k1, freq, delta, 0)
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()


@pytest.mark.parametrize("ef", [-5.0, -1.2, 0.3, 1.1])
@pytest.mark.parametrize("imag", [False, True])
def test_cut_weights_near_and_far(rp, ctx, ef, imag):
    print(f"[weights] metal ef={ef} imag={imag}", flush=True)
    kmesh, iq = (3, 2, 2), (0, 1, 0)
    rng = np.random.default_rng(9)
    E = np.sort(rng.uniform(-3.0, 3.0, 7))[None, :] + rng.uniform(-0.6, 0.6, (12, 7))
    freq = 1j * np.linspace(0.0, 9.0, 5) if imag else np.linspace(0.0, 6.0, 5) + 0j
    delta = 0.0 if imag else 0.1
    rp.rp_set_fermi_level(ctx, ef)
    got = _weights(rp, ctx, kmesh, iq, E, None, (0, 5), (2, 7), 12, freq, delta, rp.RP_W_TETRA_METAL)
    want = metal.weights_metal(kmesh, iq, E, None, 0, 5, 2, 7, 0, 12, freq, delta, ef)
    assert np.abs(got - want).max() <= 1e-11 * max(np.abs(want).max(), 1e-30)
