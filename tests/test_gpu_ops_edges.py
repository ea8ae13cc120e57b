"""The bf16 operators' newer paths at the edges of their rules, with the checks
and bars of test_gpu_ops_bf16: 3x3 convolutions whose rows come from a halo in
LDS (128- and 256-row tiles with a remainder, odd sides, tiles across images,
the widest image whose halo fits and the first that does not, 7 x 7 of 512
channels), products of one k slice, partial sums around the rules on slices, columns
and counts, and batch-norm sums of few and many rows and odd channel
counts."""
import numpy as np
import pytest
import torch

import test_gpu_ops_bf16 as base

pytestmark = pytest.mark.gpu

HALO = {
    # name: (n, h, ci, co, r, s)
    "rows128_odd": (6, 53, 64, 64, 3, 1),
    "rows256_odd": (24, 53, 64, 64, 3, 1),
    "rows128x128": (23, 27, 128, 128, 3, 1),
    "widest_halo": (20, 29, 128, 128, 3, 1),
    "past_widest": (19, 30, 128, 128, 3, 1),
    "s4_odd": (3, 7, 512, 512, 3, 1),
}


@pytest.mark.parametrize("case", list(HALO))
def test_conv_halo(case, monkeypatch):
    monkeypatch.setitem(base.CONV, case, HALO[case])
    base.test_conv_fwd_stats(case)
    base.test_conv_dgrad(case, "bnbwd")


@pytest.mark.parametrize("m", [16384, 16401])
def test_one_slice_product(m, monkeypatch):
    monkeypatch.setitem(base.DENSE, "one_slice", (m, 64, 256))
    base.test_gemm_1x1_fwd_stats("one_slice")
    monkeypatch.setitem(base.DENSE, "one_slice", (m, 256, 64))
    base.test_gemm_1x1_dgrad("one_slice", "addmask")


SUMS = [(nb, count) for count in (32768, 36866, 40004) for nb in (1, 16, 17, 32, 56)]
SUMS += [(255, 32772), (256, 32772), (40, 262140), (40, 262144), (19, 262146), (70, 300004)]


@pytest.mark.parametrize("nb,count", SUMS)
def test_sum_partials(nb, count):
    K = base._K()
    print(f"[op sum partials] {nb} x {count}", flush=True)
    part = np.random.default_rng(41).standard_normal((nb, count)).astype(np.float32)
    out = torch.full((count,), float("nan"), dtype=torch.float32, device=base.DEV)
    K.op_sum_partials(base.df(part), nb, count, out)
    # sixteen slices' sums, each in order, then the slices in order
    ref = np.zeros(count, np.float32)
    for k in range(16):
        s = np.zeros(count, np.float32)
        for b in range(k, nb, 16):
            s += part[b]
        ref += s
    assert np.array_equal(base.host(out), ref)


@pytest.mark.parametrize("nb", [1, 32, 33, 127, 129, 784, 1024, 1025, 1568])
@pytest.mark.parametrize("j", [8, 13, 64, 66, 512])
def test_bn_finalize_rows(nb, j):
    K = base._K()
    print(f"[op bn finalize] {nb} rows, {j} channels", flush=True)
    rng = np.random.default_rng(42)
    part = np.stack([rng.standard_normal((nb, j)), 2 + rng.random((nb, j))], 1)
    m = 4 * nb
    dev = torch.from_numpy(part.reshape(-1)).to(base.DEV)
    st = base.finalize_fwd(K, dev, nb, j, m)
    s1, s2 = part.sum(0)
    mean = s1 / m
    np.testing.assert_allclose(st, np.concatenate([mean, 1 / np.sqrt(s2 / m - mean ** 2 + 1e-5)]), rtol=1e-6, atol=1e-7)
    sums, dg, db = base.finalize_bwd(K, dev, nb, j, m)
    np.testing.assert_allclose(sums, np.concatenate([s1, s2]) / m, rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(db, s1, rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(dg, s2, rtol=1e-6)
