"""Small host lists copied through the pinned ring while earlier work holds the
stream: several times the ring's 4 MB of lists in calls that are queued and
not waited for, the caller's arrays overwritten after each return, and a list
larger than a segment.  With t = 0 an unfolding is a gather: every result is
compared for equality."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_queued_lists_stay_whole():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_02351_amd as rp
    ctx = rp.Context(0)
    r = np.arange(-17, 18)
    allm = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3).astype(np.int32)
    cell, W, t = rp.make_cell(np.eye(3) * 7.0, (48, 48, 48), (1, 1, 1)), np.eye(3, dtype=np.int32), np.zeros(3)
    gsph = np.ascontiguousarray(allm[np.argsort((allm ** 2).sum(1), kind="stable")][1:1501])
    chi = torch.zeros(20, 1500, 1500, 2, dtype=torch.float64, device="cuda")
    inv = torch.empty_like(chi)
    sizes = [6400 + 310 * i for i in range(60)] + [40000, 7000]     # 100 to 400 KB, 640 KB, 110 KB
    coef = torch.randn(max(sizes), 2, dtype=torch.float64, device="cuda")
    outs, picks = [], []
    torch.cuda.synchronize()
    # about 18 ms of work on the stream
    rp.rp_screen_W(ctx, cell, (0, 0, 0), 1500, gsph, 20, chi, inv, None)
    for i, n in enumerate(sizes):
        rng = np.random.RandomState(i)
        src = np.ascontiguousarray(rng.permutation(allm)[:n])
        pick = rng.permutation(n)
        dst = np.ascontiguousarray(src[pick])
        out = torch.full((1, n, 2), float("nan"), dtype=torch.float64, device="cuda")
        rp.rp_unfold_coef(ctx, cell, W, t, (0, 0, 0), src, coef[:n].reshape(1, n, 2), (0, 0, 0), dst, out)
        src[:] = 0
        dst[:] = 0
        outs.append(out)
        picks.append(pick)
    rp.rp_synchronize(ctx)
    for n, pick, out in zip(sizes, picks, outs):
        want = coef[:n][torch.from_numpy(pick).cuda()]
        print(f"[pinned ring] {n} vectors", flush=True)
        assert torch.equal(out[0], want)
    ctx.close()
