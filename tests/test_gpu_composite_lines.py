"""The composite where slices do not start on cache lines: packs cut at the
lines of each slice's output (the int32 one, the fp32 one where it is alone),
with the two outputs at different places of a line, planes smaller than a
line, grids smaller than a pack, spans of slices of every length, and the
16-bit static copy.  The int32 result is unique and compared exactly; the
fp32 field is a correctly rounded root of it and one multiplication, compared
with the oracle's at its 1e-6."""
import numpy as np
import pytest

import oracle
import scenegen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dims,n,shift_i,shift_f,copy", [
    ((1, 1, 1), 3, 0, 0, 0), ((3, 2, 5), 4, 1, 2, 0), ((31, 1, 3), 5, 0, 5, 2),
    ((16, 2, 9), 3, 0, 0, 0),    # a plane of exactly one line
    ((11, 3, 40), 7, 31, 0, 0),  # planes of 33 pixels
    ((64, 64, 8), 3, 0, 0, 0),   # aligned
    ((64, 64, 8), 3, 4, 4, 2), ((64, 64, 8), 3, 32, 7, 0),
    ((33, 27, 21), 12, 0, 0, 0), ((33, 27, 21), 12, 29, 3, 2),
    ((130, 70, 9), 11, 0, 12, 0), ((255, 9, 13), 6, 17, 17, 0),
    ((60, 52, 5), 70, 0, 8, 0)])
@pytest.mark.parametrize("outputs", ["both", "ssq", "sdf"])
def test_any_line_offset(dev, dims, n, shift_i, shift_f, copy, outputs):
    import paper_2201_05058_amd as pc
    print(f"lines {dims} n={n} +{shift_i}/+{shift_f} copy={copy} {outputs}",
          flush=True)
    sc = scenegen.small_scene(sum(dims) + n, *dims, h=0.05, n_boxes=3,
                              n_humans=2, n_slices=n)
    g = sc.grid
    rs, _ = oracle.build_static(g, sc.occ)
    wc, wf = oracle.predicted_composite(g, rs, sc.human_xy, sc.radius,
                                        sc.height)
    cnt, guard = n * g.nvox, 64
    S = torch.from_numpy(rs).to(dev)
    bufs, views = [], []
    for dtype, shift in ((torch.int32, shift_i), (torch.float32, shift_f)):
        b = torch.full((cnt + shift + guard,), 77, dtype=dtype, device=dev)
        bufs.append((b, shift))
        views.append(b[shift:shift + cnt].view((n,) + g.shape_zyx))
    h = pc.Handle()
    try:
        h.set_tuning({"composite_static16": copy})
        for G, order in ((0, 0), (1, 0), (3, 1), (n, 0)):
            h.set_tuning({"composite_static16": copy,
                          "composite_slices_per_block": G,
                          "composite_order": order})
            for b, _ in bufs:
                b.fill_(77)
            pc.predicted_composite_sdf(
                g, S, sc.human_xy, sc.radius, sc.height,
                out_ssq=views[0] if outputs != "sdf" else None,
                out_sdf=views[1] if outputs != "ssq" else None,
                want_ssq=outputs != "sdf", want_sdf=outputs != "ssq",
                handle=h)
            if outputs != "sdf":
                np.testing.assert_array_equal(views[0].cpu().numpy(), wc)
            if outputs != "ssq":
                np.testing.assert_allclose(views[1].cpu().numpy(), wf,
                                           rtol=1e-6, atol=0)
            for (b, shift), used in zip(bufs, (outputs != "sdf",
                                               outputs != "ssq")):
                v = b.cpu().numpy()  # nothing outside the view is written
                assert (v[:shift] == 77).all() and (v[shift + cnt:] == 77).all()
                assert used or (v == 77).all()
    finally:
        h.close()


@pytest.mark.parametrize("tuning", [{}, {"batch_slices_per_item": 3},
                                    {"batch_chunk_quads": 512,
                                     "batch_blocks_per_cu": 2}])
def test_batch_of_uneven_line_offsets(dev, tuning):
    import paper_2201_05058_amd as pc
    scenes, want = [], []
    for q, (dims, n, shift) in enumerate([
            ((1, 1, 1), 2, 1), ((33, 27, 21), 11, 5), ((64, 64, 8), 3, 0),
            ((64, 64, 8), 3, 8), ((11, 3, 40), 7, 31), ((50, 50, 30), 13, 0)]):
        sc = scenegen.small_scene(90 + q, *dims, h=0.05, n_boxes=3,
                                  n_humans=2, n_slices=n)
        g = sc.grid
        rs, _ = oracle.build_static(g, sc.occ)
        want.append(oracle.predicted_composite(g, rs, sc.human_xy, sc.radius,
                                               sc.height))
        buf = torch.zeros(2 * n * g.nvox + 64, dtype=torch.int32, device=dev)
        oc = buf[shift:shift + n * g.nvox].view((n,) + g.shape_zyx)
        of = buf[shift + n * g.nvox:shift + 2 * n * g.nvox].view(
            torch.float32).view((n,) + g.shape_zyx)
        scenes.append({"grid": g, "static_ssq": torch.from_numpy(rs).to(dev),
                       "human_xy": sc.human_xy, "radius": sc.radius,
                       "height": sc.height, "out_ssq": oc, "out_sdf": of})
    h = pc.Handle()
    try:
        h.set_tuning(tuning)
        for (oc, of), (wc, wf) in zip(
                pc.predicted_composite_sdf_batch(scenes, handle=h), want):
            np.testing.assert_array_equal(oc.cpu().numpy(), wc)
            np.testing.assert_allclose(of.cpu().numpy(), wf, rtol=1e-6,
                                       atol=0)
    finally:
        h.close()
