"""The pinned ring that small host lists are copied through: a segment is
written again only after the copies out of it have been read, and a list
larger than a segment is copied from the caller's memory.  On the stand-in
for the HIP runtime, which reads a queued copy as late as the library's waits
allow and counts those whose source has changed by then."""

import hip_stand_in


def test_segments_are_reused_after_their_copies(tmp_path):
    run = hip_stand_in.build(tmp_path)
    # 60 lists of 16 bytes a vector: 100 to 400 KB, in all several times the ring's 4 MB, then one of 640 KB
    first, pending, n60, small, large, bad = run(
        "hip.stand_in(Z(1 << 40), hook)\n"
        "W, t, ik = (I * 9)(1, 0, 0, 0, 1, 0, 0, 0, 1), (D * 3)(0, 0, 0), (I * 3)(0, 0, 0)\n"
        "r = np.arange(-17, 18)\n"
        "allm = np.stack(np.meshgrid(r, r, r, indexing='ij'), -1).reshape(-1, 3).astype(np.int32)\n"
        "def unfold(n, seed):\n"
        "    a = np.ascontiguousarray(np.random.RandomState(seed).permutation(allm)[:n])\n"
        "    st = rp.rp_unfold_coef(ctx, ctypes.byref(cell(48, (1, 1, 1))), W, t, ik, 1, n, ptr(a), big, L(n), ik, n, ptr(a), big, L(n))\n"
        "    a[:] = 0\n"
        "    return st\n"
        "out.append(unfold(20000, 99)); out.append(hip.stand_in_pending())\n"
        "n60 = [unfold(6400 + 310 * i, i) for i in range(60)]\n"
        "out.append(max(n60)); out.append(hip.stand_in_copies())\n"
        "unfold(40000, 7); out.append(hip.stand_in_copies())\n"
        "hip.hipStreamSynchronize(None); out.append(hip.stand_in_bad())\n")
    assert first == 0 and n60 == 0
    assert pending == 1                 # queued, not waited for
    assert small == 61 and large == 61  # every small list went through the ring, the large one did not
    assert bad == 0
