"""The per-class timing counts every launch of a gradient."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stack", [0, 2])
@pytest.mark.parametrize("n", [64, 128])
def test_the_gradient_s_probe_reduction_is_counted(n, stack):
    """Below 128 points the probe gather and its reduction, from there on the reduction of the inverse rows' sums:
    class 4, once a stack."""
    import paper_2008_11511_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-case] timing classes of a gradient n={n} stack={stack}", flush=True)
    dev, j, k, shape = torch.device("cuda:0"), 5, 2, (n + 9, n + 9)
    offs = np.random.default_rng(n).integers(0, 9, (j, 2)).astype(np.int32)
    plan = P.Plan(offs, torch.ones((j, n, n), device=dev), None, k, shape, stack=stack)
    obj = torch.ones(shape, dtype=torch.complex64, device=dev)
    probe = torch.ones((k, n, n), dtype=torch.complex64, device=dev)
    plan.timing(True)
    plan.ml_grad(obj, probe)
    stacks = -(-j // stack) if stack else 1
    per = plan.timing_read()
    for name in ("rows_fwd", "cols", "rows_inv", "gather_obj", "gather_probe"):
        assert per[name][1] == stacks, (name, per[name])
    assert per["gather_probe"][0] > 0.0
