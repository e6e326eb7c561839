"""The FP64 contraction at the edges of its tiles and slices, against the sum
of Eq. chi in torch (complex128).

Tolerance: a sum of P products in FP64 differs from the exact one by at most
about (P + 8) 2^-53 sum_p |w_p| |M_p(G)| |M_p(G')|, in the kernel and in the
reference alike; the element-wise bound here is four times that.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HA = 27.211386245988


@pytest.fixture(scope="module")
def rp():
    import paper_2001_02351_amd as rp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rp.load()
    return rp


@pytest.fixture(scope="module")
def ctx(rp):
    c = rp.Context(0)
    yield c
    c.close()


# one row / one pair; below, at and above the tile widths 32, 48, 64 and 80;
# several row tiles; pairs below one chunk, unsliced and cut into slices
@pytest.mark.parametrize("ng, nocc, nemp, nfreq", [
    (1, 1, 1, 1), (15, 1, 3, 2), (32, 4, 5, 3), (33, 8, 16, 1), (48, 3, 7, 4), (64, 17, 31, 2), (65, 9, 11, 5),
    (80, 40, 64, 3), (97, 16, 63, 2), (211, 24, 50, 7), (340, 16, 16, 1)])
@pytest.mark.parametrize("imag", [False, True])
def test_fp64_contraction_shapes(ctx, rp, ng, nocc, nemp, nfreq, imag):
    print(f"[chi f64] ng={ng} pairs={nocc * nemp} nfreq={nfreq} imag={imag}", flush=True)
    rng = np.random.default_rng([ng, nocc, nfreq, int(imag)])
    g = torch.Generator(device="cuda").manual_seed(7 * ng + nfreq)
    nb, P = nocc + nemp, nocc * nemp
    energy = torch.from_numpy(np.concatenate([rng.uniform(-8, -1, nocc), rng.uniform(1, 20, nemp)])).cuda()
    freq = 1j * np.linspace(0.0, 30.0, nfreq) if imag else np.linspace(0.0, 20.0, nfreq) + 0j
    delta = 0.0 if imag else 0.1
    M = torch.randn(P, ng, 2, generator=g, device="cuda", dtype=torch.float64)
    cell = rp.make_cell(np.eye(3) * 7.0, (16, 16, 16), (1, 1, 1))
    start = torch.randn(nfreq, ng, ng, 2, generator=g, device="cuda", dtype=torch.float64)
    if imag:   # accumulation is onto a Hermitian chi
        z = torch.view_as_complex(start)
        start = torch.view_as_real(z + z.mH).contiguous()
    e = (energy[nocc:, None] - energy[None, :nocc]).reshape(-1) / HA
    f = torch.from_numpy(freq).cuda() / HA
    w = 2.0 * (1.0 / (f[:, None] + 1j * delta / HA - e) + 1.0 / (-f[:, None] + 1j * delta / HA - e))
    Mc = torch.view_as_complex(M)
    for accumulate in (0, 1):
        chi = start.clone() if accumulate else torch.full_like(start, float("nan"))
        rp.rp_chi0_accumulate(ctx, cell, (0, 0, 0), nb, energy, None, 0, nocc, nocc, nb, 0, 1, ng, M, nfreq, freq,
                              delta, rp.RP_W_SAMPLING, rp.RP_FP64, accumulate, chi)
        rp.rp_synchronize(ctx)
        got = torch.view_as_complex(chi)
        for n in range(nfreq):
            want = (Mc.T * w[n]).contiguous() @ Mc.conj()
            size = (Mc.abs().T * w[n].abs()).contiguous() @ Mc.abs()
            if accumulate:
                want, size = want + torch.view_as_complex(start)[n], size + torch.view_as_complex(start)[n].abs()
            bound = 4.0 * (P + 8) * 2.0 ** -53 * size
            assert bool(((got[n] - want).abs() <= bound).all())
        if imag:
            assert torch.equal(got.real, got.real.mT)
