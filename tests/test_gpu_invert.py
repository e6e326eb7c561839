"""The blocked inversion at the edges of its panels, register blocks and row
counts, on matrices whose pivots lie far from the diagonal.

Tolerance: Gauss-Jordan with partial pivoting leaves a residual A X - I of
about n u |A| |X| (u = 2^-53, Frobenius norms; the growth of partial pivoting
on these random matrices is below ten); the bound is 16 n u |A| |X|.
"""

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


def _gvectors(n):
    r = int(np.ceil((n / 4.0) ** (1 / 3))) + 2
    a = np.arange(-r, r + 1)
    m = np.stack(np.meshgrid(a, a, a, indexing="ij"), -1).reshape(-1, 3)
    return np.ascontiguousarray(m[np.argsort((m ** 2).sum(1), kind="stable")][1:n + 1].astype(np.int32))


# the panel's 64 columns, the 16-, 8-, 4- and 3-column steps, the row counts
# where the threads and rows per thread change
@pytest.mark.parametrize("ng, nfreq", [
    (1, 3), (2, 1), (15, 2), (16, 1), (17, 2), (63, 1), (64, 2), (65, 1), (81, 2), (128, 1), (130, 3), (256, 1),
    (257, 2), (512, 1), (513, 1), (1024, 1), (1025, 2), (1536, 1), (1537, 1), (2048, 1), (2049, 1), (3072, 1),
    (3073, 1), (4096, 1), (4097, 1), (6143, 1),
    # 2, 3 and 4 row tiles per workgroup of the update, the last run short
    (777, 5), (517, 16), (460, 28)])
def test_inverse_with_distant_pivots(ctx, rp, ng, nfreq):
    print(f"[invert] ng={ng} nfreq={nfreq}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(ng)
    gsph = _gvectors(ng)
    lat = np.eye(3) * 7.0
    v = torch.from_numpy(np.sqrt(4 * np.pi / 343.0) / np.linalg.norm(gsph * (2 * np.pi / 7.0), axis=1)).cuda()
    # a shuffled diagonal of 2 in a random matrix of norm about one
    eps = torch.complex(*(torch.randn(nfreq, ng, ng, generator=g, device="cuda", dtype=torch.float64) / (2 * ng) ** 0.5
                          for _ in range(2)))
    for f in range(nfreq):
        eps[f, torch.randperm(ng, generator=g, device="cuda"), torch.arange(ng, device="cuda")] += 2.0
    eye = torch.eye(ng, device="cuda", dtype=torch.complex128)
    s = v[:, None] * v[None, :]
    chi = torch.view_as_real((eye - eps) / s).contiguous()
    inv = torch.full_like(chi, float("nan"))
    rp.rp_screen_W(ctx, rp.make_cell(lat, (16, 16, 16), (1, 1, 1)), (0, 0, 0), ng, gsph, nfreq, chi, inv, None)
    rp.rp_synchronize(ctx)
    for f in range(nfreq):
        a, x = eye - s * torch.view_as_complex(chi)[f], torch.view_as_complex(inv)[f]
        res = torch.linalg.norm(a @ x - eye)
        assert float(res) <= 16 * ng * 2.0 ** -53 * float(torch.linalg.norm(a) * torch.linalg.norm(x))


def test_zero_pivot_inside_a_panel_is_reported(ctx, rp):
    ng = 100
    gsph = _gvectors(ng)
    v = torch.from_numpy(np.sqrt(4 * np.pi / 343.0) / np.linalg.norm(gsph * (2 * np.pi / 7.0), axis=1)).cuda()
    chi = torch.zeros(1, ng, ng, 2, dtype=torch.float64, device="cuda")
    chi[0, 70, 70, 0] = 1.0 / float(v[70] * v[70])     # eps_70,70 = 0
    inv = torch.empty_like(chi)
    rp.rp_screen_W(ctx, rp.make_cell(np.eye(3) * 7.0, (16, 16, 16), (1, 1, 1)), (0, 0, 0), ng, gsph, 1, chi, inv, None)
    with pytest.raises(rp.RpError) as e:
        rp.rp_synchronize(ctx)
    assert e.value.status == 7
