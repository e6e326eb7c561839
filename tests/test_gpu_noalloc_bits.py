"""rp_chi0_accumulate_noalloc gives rp_chi0_accumulate's chi in every bit: both
add the pairs' terms in the same grouping, whatever room either has for
partial sums.  The sizes are those where that room differs: partial sums of
all frequencies beyond the fixed 128 MiB, weights that fill nearly all of it,
and small calls on either side of the first slice."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


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


def _call(rp, npair, ng, nfreq, imag, seed):
    """The arguments of a contraction of one occupied with npair empty bands, random M."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    M = torch.randn(npair, ng, 2, generator=g, device="cuda", dtype=torch.float64)
    energy = torch.cat([torch.zeros(1), torch.linspace(1.0, 40.0, npair)]).to("cuda", torch.float64)
    freq = 1j * np.linspace(0.1, 60.0, nfreq) if imag else np.linspace(0.0, 45.0, nfreq) + 0j
    cell = rp.make_cell(np.eye(3) * 7.0, (16, 16, 16), (1, 1, 1))
    return (cell, (0, 0, 0), 1 + npair, energy, None, 0, 1, 1, 1 + npair, 0, 1, ng, M, nfreq, freq,
            0.0 if imag else 0.1, rp.RP_W_SAMPLING)


@pytest.mark.parametrize("npair, ng, nfreq, imag", [
    (2400, 300, 20, False), (2400, 300, 21, True), (6000, 200, 20, False), (419000, 16, 20, False),
    (8300000, 2, 1, False), (127, 65, 3, False), (129, 65, 3, False)])
def test_noalloc_sums_like_the_allocating_call(ctx, rp, npair, ng, nfreq, imag):
    args = _call(rp, npair, ng, nfreq, imag, npair + ng)
    print(f"[noalloc bits] pairs={npair} ng={ng} nfreq={nfreq} imag={imag}", flush=True)
    for accumulate in (0, 1):
        a = torch.ones(nfreq, ng, ng, 2, dtype=torch.float64, device="cuda")
        b = a.clone()
        rp.rp_chi0_accumulate(ctx, *args, rp.RP_FP64, accumulate, a)
        rp.rp_chi0_accumulate_noalloc(ctx, *args, rp.RP_FP64, accumulate, b)
        rp.rp_synchronize(ctx)
        assert float(a.abs().max()) > 0.0
        assert torch.equal(a, b)
