"""Unfolding onto a target list that is a small part of the source list: no
slower than the part itself asks for, and right on either side of the rule
that sends source rows through LDS (512 source vectors, four fifths of them
picked, two rows' worth of LDS per CU).

Values: the gather and phases of Eq. symeps to 1e-14 of the largest value (one
complex product of phases and one of the element, a few roundings).  Time: the
400 inner vectors of an 8 000-vector source against those of a 400-vector
source, the same number of elements picked and written; reading whole source
rows would take twenty times the bytes of the 2 MB result (measured then: 3.9
times as long; picked: 1.0)."""

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


def _lists(ng_src, ng, inner):
    rng = np.random.default_rng(ng_src + ng)
    s = np.arange(-12, 13)
    allg = np.stack(np.meshgrid(s, s, s, indexing="ij"), -1).reshape(-1, 3)
    gi = allg[np.argsort((allg ** 2).sum(1), kind="stable")][:ng_src] if inner else rng.permutation(allg)[:ng_src]
    pick = rng.permutation(ng if inner else ng_src)[:ng]
    W, t = np.array([[0, 1, 0], [0, 0, 1], [1, 0, 0]]), np.array([0.5, 0.25, 1.0 / 3.0])
    return np.ascontiguousarray(gi.astype(np.int32)), pick, np.ascontiguousarray((gi[pick] @ W.T).astype(np.int32)), W, t


@pytest.mark.parametrize("ng_src, ng", [(511, 511), (512, 512), (640, 512), (641, 512), (4096, 4096), (4097, 4097),
                                        (4200, 3600)])
def test_both_routes(rp, ng_src, ng):
    print(f"[unfold route] ng_src={ng_src} ng={ng}", flush=True)
    gi, pick, gt, W, t = _lists(ng_src, ng, False)
    g = torch.Generator(device="cuda").manual_seed(ng_src)
    src = torch.randn(1, ng_src, ng_src, 2, generator=g, device="cuda", dtype=torch.float64)
    dst = torch.full((1, ng, ng, 2), float("nan"), dtype=torch.float64, device="cuda")
    ctx = rp.Context(0)
    rp.rp_unfold_eps_inv(ctx, rp.make_cell(np.eye(3) * 7.0, (16,) * 3, (2, 2, 2)), W, t, (0, 0, 0), gi, (0, 0, 0), gt, src,
                         dst)
    rp.rp_synchronize(ctx)
    a = gt @ t
    p = torch.from_numpy(np.exp(2j * np.pi * (a - np.floor(a)))).cuda()    # whole turns off: exp of 100 rad is off by 1e-14
    at = torch.from_numpy(pick).cuda()
    want = torch.view_as_complex(src)[:, at][:, :, at] * p[:, None] * p.conj()[None, :]
    assert float((torch.view_as_complex(dst) - want).abs().max()) <= 1e-14 * float(want.abs().max())
    ctx.close()


def test_small_target_does_not_read_the_source_rows(rp):
    ctx, cell, ms = rp.Context(0), rp.make_cell(np.eye(3) * 7.0, (16,) * 3, (2, 2, 2)), {}
    for ng_src in (400, 8000):
        gi, _, gt, W, t = _lists(ng_src, 400, True)
        src = torch.zeros(1, ng_src, ng_src, 2, device="cuda", dtype=torch.float64)
        dst = torch.empty(1, 400, 400, 2, dtype=torch.float64, device="cuda")
        times = []
        for _ in range(20):
            rp.rp_profile(ctx, True)
            rp.rp_unfold_eps_inv(ctx, cell, W, t, (0, 0, 0), gi, (0, 0, 0), gt, src, dst)
            times.append(rp.rp_profile_read(ctx)["unfold"][0])
        ms[ng_src] = min(times)
    ctx.close()
    print(f"[unfold route] 400 of 400: {ms[400] * 1e3:.1f} us, 400 of 8000: {ms[8000] * 1e3:.1f} us", flush=True)
    assert ms[8000] < 2.5 * ms[400]
