"""Dots and norms around the size up to which one workgroup does them, against the oracle.

Bound: 1e-12 of the sum of the terms' magnitudes, as for the other sizes.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 7169, 8191, 8192, 8193])
def test_small_reductions(oracle, n):
    import paper_2112_11880_amd as hk
    from paper_2112_11880_amd.hk import zdotc_noalloc
    print("[case] reductions", n, flush=True)
    rng = np.random.default_rng(n)
    x, y = (rng.standard_normal(n) + 1j * rng.standard_normal(n) for _ in range(2))
    xd, yd = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(y).to("cuda:0")
    bound = 1e-12 * np.sum(np.abs(x) * np.abs(y))
    assert abs(hk.zdotc(xd, yd).item() - oracle.zdotc(x, y)) <= bound
    assert abs(hk.zdotu(xd, yd).item() - oracle.zdotu(x, y)) <= bound
    assert abs(hk.dznrm2(xd).item() - oracle.dznrm2(x)) <= 1e-12 * oracle.dznrm2(x)
    assert torch.equal(hk.zdotc(xd, yd), zdotc_noalloc(xd, yd, torch.empty(1, dtype=torch.complex128, device="cuda:0")))
