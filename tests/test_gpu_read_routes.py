"""The forward rows on both sides of the stack size from which the same rows
of several frames lie side by side."""
import numpy as np
import pytest

import oracle
from cases import make_problem, rel_l2, small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-4          # relative, as in the parity tests


def on_device(pb, pos=None):
    import paper_2008_11511_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    to = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0", t)  # noqa: E731
    args = to(pb.iobs, torch.float32), to(pb.mask, torch.uint8), pb.wl.n_modes, pb.wl.obj_shape
    plan = P.Plan(pb.offsets, *args) if pos is None else P.Plan.with_positions(pos, *args)
    return plan, to(pb.obj0, torch.complex64), to(pb.probe0, torch.complex64), to


@pytest.mark.parametrize("k,j", [(1, 16), (1, 17), (4, 4), (4, 5)])
def test_forward_rows_around_the_cached_stack_size(k, j):
    print(f"[gpu-case] forward rows n=512 k={k} j={j}", flush=True)
    pb = make_problem(small("ml256", n=512, k=k, j=j, obj=(560, 571), step=5.0, mask_frac=0.03), start="ml")
    plan, o, p, _ = on_device(pb)
    got = plan.icalc(o, p).cpu().numpy()
    assert rel_l2(got, oracle.simulate_intensity(pb.obj0, pb.probe0, pb.offsets)) < TOL
