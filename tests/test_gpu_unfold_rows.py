"""Unfolding of G-indexed matrices whose source rows pass through LDS and of
longer ones read from memory, a shuffled list, a source list larger than the
target's: the gather and phases of Eq. symeps to 1e-14 of the largest value
(one complex product of phases and one of the element, a few roundings)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# one vector; a ragged row block; source rows of 65 KB and 96 KB (LDS) and 176 KB (memory)
@pytest.mark.parametrize("ng_src, ng, nfreq", [(1, 1, 2), (67, 66, 3), (4100, 13, 2), (6001, 9, 1), (11000, 10, 1)])
def test_unfolded_rows(ng_src, ng, nfreq):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_02351_amd as rp
    print(f"[unfold] ng_src={ng_src} ng={ng}", flush=True)
    rng = np.random.default_rng(ng_src)
    s = np.arange(-12, 13)
    allg = np.stack(np.meshgrid(s, s, s, indexing="ij"), -1).reshape(-1, 3)
    gi = np.ascontiguousarray(rng.permutation(allg)[:ng_src].astype(np.int32))
    pick = rng.permutation(ng_src)[:ng]
    W, t = np.array([[0, 1, 0], [0, 0, 1], [1, 0, 0]]), np.array([0.5, 0.25, 1.0 / 3.0])
    gt = np.ascontiguousarray((gi[pick] @ W.T).astype(np.int32))        # S G* with S = W^-T = W
    g = torch.Generator(device="cuda").manual_seed(ng_src)
    src = torch.randn(nfreq, ng_src, ng_src, 2, generator=g, device="cuda", dtype=torch.float64)
    dst = torch.full((nfreq, ng, ng, 2), float("nan"), dtype=torch.float64, device="cuda")
    ctx = rp.Context(0)
    rp.rp_unfold_eps_inv(ctx, rp.make_cell(np.eye(3) * 7.0, (16,) * 3, (2, 2, 2)), W, t, (0, 0, 0), gi, (0, 0, 0), gt, src,
                         dst)
    rp.rp_synchronize(ctx)
    p = torch.from_numpy(np.exp(2j * np.pi * (gt @ t))).cuda()
    at = torch.from_numpy(pick).cuda()
    want = torch.view_as_complex(src)[:, at][:, :, at] * p[:, None] * p.conj()[None, :]
    assert float((torch.view_as_complex(dst) - want).abs().max()) <= 1e-14 * float(want.abs().max())
    ctx.close()
