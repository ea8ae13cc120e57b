"""The LSTM step kernels at the edges of their tiles and dispatch: the bars, plans
and bit-identity checks of test_gpu_lstm on shapes with one row, one row past a
16- and a 32-row tile, hidden sizes that leave a partial 16-column tile, k
ranges on both sides of the four / sixteen wavefront rule with fewer k steps
than wavefronts, an input of another size than the state, chunks of one step
(where the recurrent product takes its own launch), chunks that no batch of
head gradients divides, and batches on the far side of the step kernels' rules:
both directions as products with the input and state parts of z apart and as
one, and only the backward so."""
import pytest

import test_gpu_lstm as base

pytestmark = pytest.mark.gpu

EDGES = {
    "one_row": dict(T=5, batch=1, input=8, hidden=8, vocab=8, grad_chunk=2),
    "rows17": dict(T=7, batch=17, input=40, hidden=24, vocab=72, grad_chunk=3),
    "rows33_k520": dict(T=6, batch=33, input=456, hidden=64, vocab=136, grad_chunk=0),
    "hidden136": dict(T=11, batch=16, input=16, hidden=136, vocab=304, grad_chunk=10),
    "chunk1": dict(T=6, batch=5, input=24, hidden=40, vocab=56, grad_chunk=1),
    "products": dict(T=4, batch=544, input=1144, hidden=264, vocab=72, grad_chunk=3),
    "products_cat": dict(T=4, batch=192, input=704, hidden=704, vocab=40, grad_chunk=3),
    "product_backward": dict(T=4, batch=288, input=24, hidden=520, vocab=40, grad_chunk=3),
}


@pytest.mark.parametrize("case", list(EDGES))
def test_lstm_step_edges(case, monkeypatch):
    monkeypatch.setitem(base.CASES, case, dict(EDGES[case], kind="lstm", seed=75))
    base.test_lstm_step_parity_all_modes(case)


def test_kernel_timer_covers_the_step_kernels():
    """The timed family's operations are those of every product of the step: the
    gates', the recurrent part of dh, the heads' three and the weight gradients."""
    import synth
    from paper_1604_06174_amd import ckpt as K
    from paper_1604_06174_amd.workload import GpuStep
    cfg = dict(base.CASES["mid"])
    T, B, E, H, V = (cfg[k] for k in ("T", "batch", "input", "hidden", "vocab"))
    d = synth.make(cfg)
    step = GpuStep(cfg, d["params"], d["input"], d["target"])
    step.net.timing_enable(True)
    step.run(step.plan(K.NONE))
    kt = step.net.timing_read()
    step.net.timing_enable(False)
    gates = T * 8 * B * H * E + (T - 1) * 8 * B * H * H
    heads = 3 * T * 2 * B * V * H
    weights = T * 8 * B * H * (E + H)
    assert kt["flops"] == gates + (T - 1) * 8 * B * H * H + heads + weights
    assert kt["ms"] > 0 and kt["launches"] >= 2 * T
