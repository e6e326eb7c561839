"""V and X of a q-term against their definitions in 80-bit arithmetic on grids
with many planes along the first axis, whose sum must not be a chain of one
addition per plane; and a list with more vectors than one pass over them holds.

Tolerance (u = 2^-53, errors as random walks of steps 0.6 u): the constants
and the scale, in every element alike and squared, 9 roundings, 1.8 u; a
density's transform 15 roundings in each factor, 3.3 u, over the ten vectors
that make up most of a sum 1 u: 2.1 u together.  256 planes one after the
other, half of them adding to a large sum, would put 4.8 u on top of it.  The
mean over eight systems has to stay below 3.3 u."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LD, CLD = np.longdouble, np.clongdouble
PI = LD("3.14159265358979323846264338327950288")


@pytest.mark.parametrize("edge, ncell, ntail", [((256, 16, 16), 27, 0), ((256, 16, 16), 1, 0), ((128, 24, 24), 27, 900),
                                                ((256, 16, 16), 27, 2500)])
def test_many_planes(edge, ncell, ntail):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if np.finfo(LD).nmant < 63:
        pytest.skip("no 80-bit long double")
    import paper_2001_02351_amd as rp
    ctx, a0, q, nwan, ng = rp.Context(0), 7.0, np.array([0.25, 0.0, 0.0]), 3, 100
    r = np.arange(-7, 8)
    m = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
    gl = np.ascontiguousarray(m[np.argsort(((m + q) ** 2).sum(1), kind="stable")][:ng + ntail].astype(np.int32))
    cells = np.stack(np.meshgrid(*[[0, -1, 1]] * 3, indexing="ij"), -1).reshape(-1, 3)[:ncell].astype(np.int32)
    cell = rp.make_cell(np.eye(3) * a0, edge, (4, 4, 4))
    pre = LD("27.211386245988") * 4 * PI / (LD(a0) ** 3 * 64)
    eps = torch.zeros(1, ng, ng, 2, dtype=torch.float64, device="cuda")
    err = {"V": [], "X": []}
    for seed in range(8):
        rng = np.random.default_rng(seed)
        cen, phi = rng.uniform(0, 1, (nwan, 3)), np.empty((nwan,) + edge)
        for i in range(nwan):
            d = [np.arange(n) / n - c for n, c in zip(edge, cen[i])]
            f = [np.exp(-rng.uniform(0.3, 0.8) * ((x - np.floor(x + 0.5)) * a0) ** 2) for x in d]
            phi[i] = f[0][:, None, None] * f[1][None, :, None] * f[2][None, None, :]
            phi[i] /= np.sqrt((phi[i] ** 2).sum() * a0 ** 3 / phi[i].size)
        rho = np.stack([_density(phi[i], cen[i], q, gl, edge, a0) for i in range(nwan)])
        V, X = (torch.zeros(ncell, nwan, nwan, 2, dtype=torch.float64, device="cuda") for _ in range(2))
        rp.rp_wannier_qterm(ctx, cell, (1, 0, 0), nwan, torch.from_numpy(phi).cuda(), cen, cells, ng, gl[:ng].copy(), ntail,
                            gl[ng:].copy(), 1, eps, 0, None, None, V, X)
        rp.rp_synchronize(ctx)
        v0 = pre * np.array([[(rho[i] * rho[j].conj()).sum() for j in range(nwan)] for i in range(nwan)])
        got = torch.view_as_complex(V)[0].cpu().numpy()
        err["V"].append(float(np.sqrt((np.abs(got - v0) ** 2).sum() / (np.abs(v0) ** 2).sum())))
        # the overlap density of an orbital with itself in the home cell is its direct density
        x0, got = np.diag(v0), np.diag(torch.view_as_complex(X)[0].cpu().numpy())
        err["X"].append(float(np.sqrt((np.abs(got - x0) ** 2).sum() / (np.abs(x0) ** 2).sum())))
    ctx.close()
    for k, e in err.items():
        print(f"[density accuracy] {edge} cells={ncell} tail={ntail}: {k} mean {np.mean(e) * 2 ** 53:.1f} u", flush=True)
    assert max(np.mean(e) for e in err.values()) < 3.3 * 2.0 ** -53


def _density(phi, cen, q, gl, edge, a0):
    """rho_i(G) = (Omega / N_r) sum_p phi^2 e^{i (q + G).rt} / |q + G| of one orbital, axis by axis."""
    g = phi.astype(LD) ** 2
    ms = [np.unique(gl[:, a]) for a in range(3)]
    for a in range(3):
        p = np.arange(edge[a])
        rt = LD(1) * p / LD(edge[a]) - np.floor(p / edge[a] - cen[a] + 0.5).astype(LD)
        shape = [1, 1, 1]
        shape[a] = edge[a]
        g = g * np.exp(2j * PI * LD(q[a]) * rt).reshape(shape)
    for a in range(3):
        p = np.arange(edge[a])
        F = np.exp(2j * PI * ((ms[a][:, None] * p[None, :]) % edge[a]).astype(LD) / LD(edge[a])).astype(CLD)
        g = np.moveaxis(np.tensordot(F, g, (1, a)), 0, a)
    ix = [np.searchsorted(ms[a], gl[:, a]) for a in range(3)]
    qg = np.sqrt((((q.astype(LD) + gl.astype(LD)) * (2 * PI / LD(a0))) ** 2).sum(1))
    return g[ix[0], ix[1], ix[2]] * (LD(a0) ** 3 / LD(int(np.prod(edge)))) / qg
