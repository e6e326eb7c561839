"""Calls on a device that is nearly full: workspace that only speed asks for is
cut down to what there is, and a call fails with RP_E_NOMEM only without the
room that it cannot do without.  Runs on the stand-in for the HIP runtime
(hip_stand_in), which limits the memory and shows the buffers that launches
are given."""

import pytest

import hip_stand_in


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    return hip_stand_in.build(tmp_path_factory.mktemp("stand_in"))


def _chi(call):
    assert call["status"] == 0 and call["err"] == ""
    chi = [x for x in call["launches"] if x["k"] == "chi"]
    for x in chi:
        assert x["y"] == x["nslice"]
        if x["nslice"] > 1:
            assert x["need"] <= x["room"]
    assert sum(x["nfreq"] for x in chi) == 20
    assert sum(x["nfreq"] for x in call["launches"] if x["k"] == "sum") in (0, 20)
    return chi


def test_fp64_partial_sums_take_what_there_is(stand_in):
    """2 400 pairs, N_G = 300, 20 frequencies: weights 0.8 MB; partial chi of
    all frequencies 29 MB per slice.  With less room the frequencies go in
    groups with the same slices; with none the pairs are not cut."""
    full, some, none, again, no = stand_in(
        "call(400*MB, accumulate, 2400, 300, 20)\n"
        "rp.rp_destroy(ctx); rp.rp_create(ctypes.byref(ctx), 0, None); call(40*MB, accumulate, 2400, 300, 20)\n"
        "rp.rp_destroy(ctx); rp.rp_create(ctypes.byref(ctx), 0, None); call(1*MB, accumulate, 2400, 300, 20)\n"
        "call(0, accumulate, 2400, 300, 20)\n"
        "rp.rp_destroy(ctx); rp.rp_create(ctypes.byref(ctx), 0, None); call(0, accumulate, 2400, 300, 20)\n")
    slices = _chi(full)[0]["nslice"]
    assert slices > 1 and len(_chi(full)) == 1
    chi = _chi(some)
    assert len(chi) > 1 and all(x["nslice"] == slices for x in chi)
    assert [x["nslice"] for x in _chi(none)] == [1]
    assert [x["nslice"] for x in _chi(again)] == [1]        # nothing more is asked for
    assert no["status"] == 5 and not no["launches"]         # RP_E_NOMEM: no room for the weights


def _ugrids(call, bands, nk, one):
    assert call["status"] == 0 and call["err"] == ""
    u = [x for x in call["launches"] if x["k"] == "ugrid"]
    assert sum(x["n"] for x in u) == nk
    for x in u:
        assert x["bands"] == bands and x["n"] * one <= x["room"]
    return u


def test_u_grids_of_fewer_k_points(stand_in):
    """27 k-points of 12 bands on 20^3 in FP64: 1.5 MB of u-grids each, taken
    together where there is room, fewer at a time where there is not; one
    k-point's are the least.  The same in a batch, whose graphs hold the
    groups that the workspace had room for."""
    one = 16 * 12 * 20 ** 3      # the batch: M 0.8 MB, weights and partial sums beside it
    new = "rp.rp_destroy(ctx); rp.rp_create(ctypes.byref(ctx), 0, None); "
    full, some, least, no, batch, again, run = stand_in(
        "call(400*MB, pair, (3, 3, 3), 20, 4, 8, 60, 0)\n" +
        new + "call(12*MB, pair, (3, 3, 3), 20, 4, 8, 60, 0)\n" +
        new + "call(2*MB, pair, (3, 3, 3), 20, 4, 8, 60, 0)\n" +
        new + "call(1*MB, pair, (3, 3, 3), 20, 4, 8, 60, 0)\n" +
        new + "keep = []; p = problem((3, 3, 3), 20, 4, 8, 60, 20, 27, keep)\n"
        "call(16*MB, rp.rp_chi0_batch, ctx, 1, ctypes.byref(p), 0); call(0, rp.rp_chi0_batch, ctx, 1, ctypes.byref(p), 0)\n" +
        # M of 21 MB and its weights have to fit beside the grids, which were asked for first
        new + "p = problem((3, 3, 3), 20, 16, 32, 100, 20, 27, keep); call(40*MB, rp.rp_chi0_run, ctx, ctypes.byref(p), 0)\n")
    assert len(_ugrids(full, 12, 27, one)) == 1
    assert 1 < len(_ugrids(some, 12, 27, one)) < 27
    assert len(_ugrids(least, 12, 27, one)) == 27
    assert no["status"] == 5 and not no["launches"]
    assert 1 < len(_ugrids(batch, 12, 27, one)) < 27
    assert [x["k"] for x in again["launches"]] == ["graph"]
    assert 1 < len(_ugrids(run, 48, 27, 4 * one)) <= 27


def test_inversion_of_fewer_matrices(stand_in):
    """16 matrices of 300: 0.94 MB of panels and pivot rows each, all at once
    where there is room, fewer at a time where there is not."""
    one = 16 * 64 * (3 * 300 + 16)
    new = "rp.rp_destroy(ctx); rp.rp_create(ctypes.byref(ctx), 0, None); "
    full, some, least, no = stand_in("call(40*MB, screen, 300, 16)\n" + new + "call(5*MB, screen, 300, 16)\n" + new +
                                     "call(1*MB, screen, 300, 16)\n" + new + "call(MB//2, screen, 300, 16)\n")
    for call, groups in ((full, 1), (some, None), (least, 16)):
        assert call["status"] == 0 and call["err"] == ""
        gj = [x for x in call["launches"] if x["k"] == "gj"]
        assert sum(x["nmat"] for x in gj) == 16
        assert all(x["nmat"] * one <= x["room"] for x in gj)
        assert len(gj) == groups if groups else 1 < len(gj) < 16
    assert no["status"] == 5 and not no["launches"]
