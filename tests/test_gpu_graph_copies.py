"""A captured batch whose positions change between launches that are still
running: every launch writes the fields of the positions set before it, also
those of scenes not touched since an earlier launch, on one stream and from
one stream to another."""
import numpy as np
import pytest

from test_gpu_batch import plain, ragged_scenes, scene_dict

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("streams", [1, 2])
def test_positions_set_while_launches_run(dev, streams):
    import paper_2201_05058_amd as pc
    scs = ragged_scenes(40)
    ds = [scene_dict(pc, sc, dev) for sc in scs]
    base = [np.array(sc.human_xy) for sc in scs]
    move = [i for i, b in enumerate(base) if b.size]
    g = pc.BatchGraph(ds)
    ss = [torch.cuda.Stream(dev) for _ in range(streams)]
    torch.cuda.synchronize()
    # scenes moved before each launch, and whether all move
    plan = [[], move[:1], move[1:3], [], move[:2], move, move[-1:], [], move]
    got, want, prev = [], [], None
    for step, scenes in enumerate(plan):
        for q in scenes:
            xy = base[q] + 0.07 * (step + 1) * np.array([1.0, -0.6])
            g.set_positions(q, xy)
            ds[q]["human_xy"] = xy
        want.append([d["human_xy"] for d in ds])
        s = ss[step % streams]
        if prev is not None:  # the copies below read the outputs first
            s.wait_event(prev)
        with torch.cuda.stream(s):
            g.launch()
            got.append([(c.clone(), f.clone()) for c, f in g.outputs])
            prev = torch.cuda.Event()
            prev.record(s)
    torch.cuda.synchronize()
    for step, (outs, xys) in enumerate(zip(got, want)):
        print("graph copies: launch", step, flush=True)
        for d, xy, (c, f) in zip(ds, xys, outs):
            rc, rf = plain(pc, {**d, "human_xy": xy})
            assert torch.equal(c, rc) and torch.equal(f, rf)
    g.close()
