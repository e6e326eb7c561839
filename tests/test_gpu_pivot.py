"""The pivot of the inversion is the entry of largest modulus, not of largest
|re| + |im|: a column whose only entry above the reported floor (1e-13) is
real, beside one of larger |re| + |im| whose modulus is below the floor, is
inverted and not reported as singular.

With a = 1.2e-13 and b = 0.68e-13 (1 + i) the block [[a, 1], [b, d]], d of
the size of rounding, has the inverse [[., 1/b], [1, .]] to terms of 1e-15
relative; the elimination adds a few roundings, and eps from chi one (1e-13 is
left for all of them)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# the block in the first and the last columns, two of the register shapes of the steps
@pytest.mark.parametrize("ng, c", [(2, 0), (300, 0), (300, 298), (700, 611), (1100, 0)])
def test_pivot_by_modulus(ng, c):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_02351_amd as rp
    print(f"[pivot] ng={ng} c={c}", flush=True)
    r = np.arange(-8, 9)
    m = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
    gsph = np.ascontiguousarray(m[np.argsort((m ** 2).sum(1), kind="stable")][1:ng + 1].astype(np.int32))
    v = torch.from_numpy(np.sqrt(4 * np.pi / 343.0) / np.linalg.norm(gsph * (2 * np.pi / 7.0), axis=1)).cuda()
    eye = torch.eye(ng, device="cuda", dtype=torch.complex128)
    eps, b = eye.clone(), 0.68e-13 * (1 + 1j)
    eps[c, c], eps[c + 1, c], eps[c, c + 1], eps[c + 1, c + 1] = 1.2e-13, b, 1.0, 0.0
    chi = torch.view_as_real((eye - eps) / (v[:, None] * v[None, :]))[None].contiguous()
    inv = torch.full_like(chi, float("nan"))
    ctx = rp.Context(0)
    rp.rp_screen_W(ctx, rp.make_cell(np.eye(3) * 7.0, (16, 16, 16), (1, 1, 1)), (0, 0, 0), ng, gsph, 1, chi, inv, None)
    rp.rp_synchronize(ctx)      # raises where a pivot below the floor was taken
    x = torch.view_as_complex(inv)[0]
    assert abs(complex(x[c, c + 1]) * b - 1.0) < 1e-13
    assert abs(complex(x[c + 1, c]) - 1.0) < 1e-13
    ctx.close()
