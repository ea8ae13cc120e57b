"""The residual MLP's products at the edges of their tiles and dispatch: the bars,
plans and bit-identity checks of test_gpu_mlp on one row, widths that are no
multiple of the 4-float loads, of the 16-wide k groups or of the 128-wide k
slices, k ranges shorter than the wavefronts that share them, more rows than one
workgroup sums for a bias gradient (and more than it sums last), a product of 64 x
64 tiles, and both sides of the rule by which a backward's products run one by
one; and the node graph's step (which runs the products unfused) against the chain's."""
import pytest

import synth
import test_gpu_mlp as base

pytestmark = pytest.mark.gpu

EDGES = {
    "one_row": dict(depth=3, width=3, batch=1),
    "w33": dict(depth=5, width=33, batch=31),
    "w130": dict(depth=5, width=130, batch=33),
    "w132": dict(depth=5, width=132, batch=65),
    "w300": dict(depth=3, width=300, batch=200),
    "rows1025": dict(depth=3, width=36, batch=1025),
    "tiles64": dict(depth=2, width=512, batch=2048),
    "rows513": dict(depth=3, width=72, batch=513),
    # both sides of the rules, vectors and not; two million ReLU decisions: each case's first seed
    # from 57 on for which the oracle's float64 run has every one at least three times the
    # root-mean-square error of its float32 run from zero
    "before_products": dict(depth=2, width=1028, batch=1016, seed=62),
    "products": dict(depth=2, width=1028, batch=1017, seed=75),
    "products_odd": dict(depth=2, width=1025, batch=1023, seed=57),
    "products_rows": dict(depth=2, width=452, batch=452, seed=57),
}


@pytest.mark.parametrize("case", list(EDGES))
def test_mlp_step_edges(case, monkeypatch):
    import torch
    from paper_1604_06174_amd import ckpt as K
    from paper_1604_06174_amd.workload import GpuStep
    cfg = dict(dict(kind="mlp", seed=57), **EDGES[case])
    monkeypatch.setitem(base.CASES, case, cfg)
    base.test_mlp_step_parity_all_modes(case)
    d = synth.make(cfg)
    step = GpuStep(cfg, d["params"], d["input"], d["target"])
    step.grads.fill_(float("nan"))  # the gaps between parameters keep it
    step.run(step.plan(K.NONE))
    torch.cuda.synchronize()
    chain = step.grads_bytes()
    step.grads.fill_(float("nan"))
    step.run_graph(step.graph_plan())
    torch.cuda.synchronize()
    assert step.grads_bytes() == chain
