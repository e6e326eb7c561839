"""The weights that the split contractions use at complex frequencies: every
tetrahedron's divided difference by itself, in the kernel of insulators and in
that of metals alike.  With the Fermi level in the gap no tetrahedron is cut,
and chi of the two weight modes is the same in every bit.

M is the identity (as many vectors as pairs), so that a diagonal element of
chi is one weight, rounded to the FP32 value that the six-product form keeps
whole (2^-22 |w| is left for it): a weight that differs in its 14th digit
shows in about one of a million roundings, more where the frequencies lie
between the corners' energies with little broadening, as here."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_insulating_and_metallic_kernels_give_the_same_chi():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_02351_amd as rp
    ctx = rp.Context(0)
    km, nocc, nemp, nfreq, delta = (4, 4, 4), 4, 6, 50, 0.005
    nk, nb, P = 64, nocc + nemp, 64 * nocc * nemp
    cell = rp.make_cell(np.eye(3) * 7.0, (16, 16, 16), km)
    k = np.stack(np.meshgrid(*[np.arange(n) / n for n in km], indexing="ij"), -1).reshape(-1, 3)
    M = torch.zeros(P, P, 2, dtype=torch.float64, device="cuda")
    M[torch.arange(P), torch.arange(P), 0] = 1.0
    chi = [torch.empty(nfreq, P, P, 2, dtype=torch.float64, device="cuda") for _ in range(2)]
    w = torch.empty(nfreq, P, 2, dtype=torch.float64, device="cuda")
    rp.rp_set_fermi_level(ctx, 0.0)
    other = 0
    for seed in range(6):
        rng = np.random.default_rng(seed)
        c = np.concatenate([rng.uniform(-14, -4, nocc), rng.uniform(4, 24, nemp)])
        a = rng.uniform(-1, 1, (3, nb))
        E = c[None] + 3.0 * (np.cos(2 * np.pi * k) @ a) / np.abs(a).sum(0)
        assert E[:, :nocc].max() < 0.0 < E[:, nocc:].min()
        energy = torch.from_numpy(np.ascontiguousarray(E)).cuda()
        freq = np.linspace(0.0, 40.0, nfreq) + 0j
        args = (cell, (1, 0, 0), nb, energy, None, 0, nocc, nocc, nb, 0, nk)
        for x, mode in zip(chi, (rp.RP_W_TETRA, rp.RP_W_TETRA_METAL)):
            rp.rp_chi0_accumulate(ctx, *args, P, M, nfreq, freq, delta, mode, rp.RP_SPLIT_BF16_X6, 0, x)
        rp.rp_weights(ctx, *args, nfreq, freq, delta, rp.RP_W_TETRA, w)
        rp.rp_synchronize(ctx)
        assert torch.equal(chi[0], chi[1])
        d = torch.diagonal(chi[0], dim1=1, dim2=2).transpose(1, 2)      # [nfreq][P][2]
        assert bool(((d - w).abs() <= 2.0 ** -22 * w.abs()).all())
        other += int((d.float() != w.float()).sum())
    print(f"[split weight bits] {6 * w.numel()} values, {other} of them rounded otherwise than rp_weights' would be", flush=True)
    ctx.close()
