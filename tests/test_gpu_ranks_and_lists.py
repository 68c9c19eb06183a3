"""GPU: every r_b of the batched tail, and the chunking of the training lists.

The tail is compiled per r_b (0 to 8) and the covariance takes its training
vectors in whole chunks of 16 with a half chunk for a remainder of 1 to 8, so
the ranks and the remainders at the edges are run against the FP64 oracle, as
a frame (sliding window: the entering and leaving lists) and as a probe (the
full list).
"""
import numpy as np
import pytest

import oracle
import scenegen

pytestmark = pytest.mark.gpu

BAR = {"fp32": 1e-4, "bf16x3": 5e-6, "fp32_f64": 1e-6}   # the paths' accuracy on clutter scenes
RANKS = [(q, rb, "fp32") for q in (8, 12, 16) for rb in range(0, 9) if (q, rb) != (8, 8)]
RANKS += [(16, rb, prec) for rb in (1, 2, 3) for prec in ("bf16x3", "fp32_f64")] + [(8, 7, "bf16x3"), (16, 8, "bf16x3")]
LISTS = [(q, n) for q in (8, 16) for n in (56, 57, 63, 64, 65, 71, 72, 73, 79, 80, 96, 255)]


def run_case(q, n, rb, precision):
    import torch

    import paper_1604_03622_amd as kstap
    spec = scenegen.SceneSpec(p=3, q=q, H=25, W=27, r_a=1, r_b=max(rb, 1), n_targets=2)
    sc = scenegen.make_scene(spec, seed=1000 * q + 10 * n + rb)
    cfg = oracle.OracleConfig(p=3, q=q, n=n, r_a=1, r_b=rb)
    ref = oracle.kron_stap_frame(sc.x, cfg)
    assert ref["pixels"].shape[0] > 0
    plan = kstap.Plan(p=3, q=q, n=n, r_a=1, r_b=rb, precision=precision)
    x = torch.from_numpy(sc.x).cuda()
    r, c = ref["pixels"][:, 0], ref["pixels"][:, 1]
    frame = kstap.run(plan, x)[0].cpu().numpy()[r, c]
    probe = kstap.probe(plan, x, ref["pixels"])["T"].cpu().numpy()
    want = ref["T_img"][r, c]
    for got in (frame, probe):
        assert np.max(np.abs(got - want) / np.maximum(want, 1.0)) <= BAR[precision]


@pytest.mark.parametrize("q,rb,precision", RANKS)
def test_every_rank(q, rb, precision):
    run_case(q, 64, rb, precision)


@pytest.mark.parametrize("q,n", LISTS)
def test_list_remainders(q, n):
    run_case(q, n, 3, "fp32")


def test_remainders_cover_the_chunking():
    """The lists above end in whole chunks and in half chunks, full and one entry over."""
    assert {n % 16 for _, n in LISTS} >= {0, 1, 7, 8, 9, 15}
