"""Serving steps on two streams with their tables read from mapped host
memory: frames cut into slices of many steps, several kernel classes in one
step, and steps with more slices than one pass of the table copy covers.  Each
result is bitwise the frame's own."""
import pytest

import scenegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,side,inflight,step", [(1, 96, 1, 0), (5, 130, 3, 4096), (90, 33, 90, 0)],
                         ids=["one", "sliced", "many"])
def test_served_steps_equal_alone(frames, side, inflight, step):
    import paper_1604_03622_amd as kstap
    plans = [kstap.Plan(p=3, q=16, n=96, r_a=1, r_b=4), kstap.Plan(p=3, q=8, n=64, r_a=1, r_b=3),
             kstap.Plan(p=3, q=16, n=96, r_a=1, r_b=3, precision="bf16x3")]
    scenes = {q: scenegen.make_scene(scenegen.SceneSpec(p=3, q=q, H=side, W=side + 3, r_b=3, n_targets=2), 70 + q)
              for q in (8, 16)}
    xs = {q: torch.from_numpy(s.x) for q, s in scenes.items()}
    alone = []
    for pl in plans:
        T, D = kstap.run(pl, xs[pl.q].cuda())
        alone.append((T.cpu(), D.cpu()))
    # a first frame that keeps the device busy while the others become ready
    big = scenegen.make_scene(scenegen.SceneSpec(p=3, q=16, H=400, W=400, r_b=3, n_targets=2), 91)
    xb = torch.from_numpy(big.x).cuda()
    Tb, Db = kstap.run(plans[0], xb)
    srv = kstap.Server(hbm_budget_bytes=1 << 30, max_inflight=inflight, step_pixels=step)
    pinned = {q: x.pin_memory() for q, x in xs.items()}
    for rnd in range(2):
        first = srv.submit(plans[0], xb)
        tickets = [srv.submit(plans[i % 3], pinned[plans[i % 3].q]) for i in range(frames)]
        T, D, _ = srv.wait(first, timeout_ms=60000)
        assert torch.equal(T, Tb.cpu()) and torch.equal(D, Db.cpu())
        for i, t in enumerate(tickets):
            T, D, _ = srv.wait(t, timeout_ms=60000)
            assert torch.equal(T, alone[i % 3][0]), f"round {rnd}, frame {i}: T differs from the frame alone"
            assert torch.equal(D, alone[i % 3][1]), f"round {rnd}, frame {i}: D differs from the frame alone"
    srv.close()
