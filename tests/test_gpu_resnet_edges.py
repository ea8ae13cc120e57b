"""GPU: the launches that form a stride-1 convolution's two gradients together
(16, 32 and 64 channels at 32, 16 and 8 pixels), at batches that leave the
weight gradient a last tile or pixel range of its own, against the float64
oracle, and with the first ReLU's output kept or formed again as it is read."""
import numpy as np
import pytest

import synth
from oracle import nets, units as U

pytestmark = pytest.mark.gpu

TOL = 1e-4  # float32 sums of up to 5,120 products; ReLU decisions checked to be clear below


def _err(g, o):
    g, o = (np.asarray(v, np.float64).reshape(-1) for v in (g, o))
    return float(np.max(np.abs(g - o)) / max(np.max(np.abs(o)), 1e-30))


# (batch, seed): seeds whose ReLU decisions float32 leaves alone.  Seed 72 at batch 3 is not one,
# although the oracle's own float32 run happens to agree there: the separate launches of the two
# gradients differ from float64 in the very bits that the joint one gives (one decision, 1.7e-2).
@pytest.mark.parametrize("batch,seed", [(1, 71), (3, 71), (5, 72)])
@pytest.mark.parametrize("drop", [0, 1])
def test_gradient_pairs_against_oracle(batch, seed, drop):
    from paper_1604_06174_amd import ckpt as K
    from paper_1604_06174_amd.workload import GpuStep
    cfg = dict(kind="resnet_basic", blocks_per_stage=2, base=16, batch=batch, image=32, classes=10, seed=seed,
               drop_bn_relu=drop)
    d = synth.make(cfg)
    _, o = nets.full_storage_step(nets.Chain(d["structure"], d["params"], U.F64), d["input"], d["target"])
    _, o32 = nets.full_storage_step(nets.Chain(d["structure"], d["params"], U.Prec(np.float32)), d["input"], d["target"])
    assert max(_err(o32[k], o[k]) for k in o) < 2e-5, "not well posed at float32"
    step = GpuStep(cfg, d["params"], d["input"], d["target"])
    print(f"[gradient pairs] batch={batch} drop={drop}", flush=True)
    step.run(step.plan(K.SQRT))
    g = step.grads_host()
    for k in o:
        assert _err(g[k], o[k]) <= TOL, (k, _err(g[k], o[k]))
