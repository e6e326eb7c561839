"""W_ij against its definition in 80-bit arithmetic: the quadratic forms over a
thousand vectors add no more rounding than a sum by halves would.

Tolerance (u = 2^-53, errors as random walks of steps 0.6 u or less): a density
takes about 15 roundings in its transform and 5 in its phases, of both
densities 40; a product of four columns 8, their sum over a row by halves (or
with its rounding errors kept) up to 10, the rows' sum 10 more: 0.6 u sqrt(68)
= 5 u; the mean over six systems has to stay below 6 u.  Chains of 400
additions alone (a quarter of the columns into one accumulator, 32 rows one
after the other) would be 12 u."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LD, CLD = np.longdouble, np.clongdouble
PI = LD("3.14159265358979323846264338327950288")


def _mm(a, b):
    out = np.zeros((a.shape[0], b.shape[1]), CLD)
    for k in range(a.shape[1]):
        out += a[:, k:k + 1] * b[k:k + 1, :]
    return out


def _density(phi, cen, q, gl, edge, a0):
    """rho_i(G) = (Omega / N_r) sum_p phi^2 e^{i (q + G).rt} / |q + G| of one orbital, axis by axis."""
    p, ms = np.arange(edge), [np.unique(gl[:, a]) for a in range(3)]
    g = phi.astype(LD) ** 2
    for a in range(3):
        x = p / edge - cen[a]
        rt = LD(1) * p / LD(edge) - np.floor(x + 0.5).astype(LD)
        shape = [1, 1, 1]
        shape[a] = edge
        g = g * np.exp(2j * PI * LD(q[a]) * rt).reshape(shape)
    for a in range(3):
        F = np.exp(2j * PI * ((ms[a][:, None] * p[None, :]) % edge).astype(LD) / LD(edge))
        g = np.moveaxis(np.tensordot(F, g, (1, a)), 0, a)
    ix = [np.searchsorted(ms[a], gl[:, a]) for a in range(3)]
    qg = np.sqrt((((q.astype(LD) + gl.astype(LD)) * (2 * PI / LD(a0))) ** 2).sum(1))
    return g[ix[0], ix[1], ix[2]] * (LD(a0) ** 3 / LD(edge) ** 3) / qg


@pytest.mark.parametrize("edge, nwan, ng", [(32, 4, 777), (32, 18, 900), (27, 3, 1100)])
def test_quadratic_forms_round_like_sums_by_halves(edge, nwan, ng):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if np.finfo(LD).nmant < 63:
        pytest.skip("no 80-bit long double")
    import paper_2001_02351_amd as rp
    ctx, a0, q = rp.Context(0), 7.0, np.array([0.25, 0.0, 0.0])
    r = np.arange(-8, 9)
    m = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
    gs = np.ascontiguousarray(m[np.argsort(((m + q) ** 2).sum(1), kind="stable")][:ng].astype(np.int32))
    cell = rp.make_cell(np.eye(3) * a0, (edge,) * 3, (4, 4, 4))
    pre = LD("27.211386245988") * 4 * PI / (LD(a0) ** 3 * 64)
    err = []
    for seed in range(6):
        rng = np.random.default_rng([seed, ng])
        cen, x = rng.uniform(0, 1, (nwan, 3)), np.arange(edge) / edge
        phi = np.empty((nwan, edge, edge, edge))
        for i in range(nwan):
            f = [np.exp(-rng.uniform(1.1, 1.9) * ((d - np.floor(d + 0.5)) * a0) ** 2) for d in (x - c for c in cen[i])]
            phi[i] = f[0][:, None, None] * f[1][None, :, None] * f[2][None, None, :]
            phi[i] /= np.sqrt((phi[i] ** 2).sum() * a0 ** 3 / edge ** 3)
        b = (rng.standard_normal((ng, 96)) + 1j * rng.standard_normal((ng, 96))) / np.sqrt(2 * ng)
        einv = np.eye(ng) - (b * (rng.random(96) * (0.6 + 0.2j))) @ b.conj().T
        e = torch.view_as_real(torch.from_numpy(einv)).contiguous().cuda()[None].contiguous()
        w = torch.empty(1, nwan, nwan, 2, dtype=torch.float64, device="cuda")
        rp.rp_wannier_W(ctx, cell, (1, 0, 0), nwan, torch.from_numpy(phi).cuda(), cen, ng, gs, 0, np.zeros((0, 3), np.int32),
                        1, e, w)
        rp.rp_synchronize(ctx)
        rho = np.stack([_density(phi[i], cen[i], q, gs, edge, a0) for i in range(nwan)])
        want = pre * _mm(_mm(rho, einv.astype(CLD)), rho.conj().T)
        got = torch.view_as_complex(w)[0].cpu().numpy()
        err.append(float(np.sqrt((np.abs(got - want) ** 2).sum() / (np.abs(want) ** 2).sum())))
    ctx.close()
    print(f"[wij accuracy] edge={edge} nwan={nwan} ng={ng}: mean {np.mean(err) * 2 ** 53:.1f} u, max {max(err) * 2 ** 53:.1f} u",
          flush=True)
    assert np.mean(err) < 6 * 2.0 ** -53
